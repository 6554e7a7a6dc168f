// Vector kernels of the Krylov solves of Newton's linear step (BiCGStab and
// restarted GMRES, gfx950): block-Jacobi preconditioner from the 4x4 diagonal
// blocks of the assembled Jacobian, deterministic inner products, combinations
// of Krylov vectors. All vectors are FP64 with 4 entries per node.
//
// They are bound by launches and waits on small systems and by HBM on large
// ones, so an update carries the inner products of its result and its
// preconditioned copy, coefficients that only the device needs stay there, and
// the host reads one set of sums per step, written into its own memory by the
// kernel that forms them. Assembly and 30 GMRES steps on 92127 nodes (FP64): 7.57
// ms with a kernel per operation and a wait per product, 5.15 ms so (4.85 ms with the
// assembly as it is now); per step
// 52 us for the matrix product (6 TB/s), 35 us for the three sweeps (16 vectors on
// average, 4.7 TB/s) and 18 us for their sums and the next vector.
#include "kernels.h"

namespace vmsk {

namespace {
constexpr int KB = 256;  // threads per block of the vector kernels

unsigned blocks_for(int64_t n, int64_t cap) {
    int64_t g = (n + KB - 1) / KB;
    if (g > cap) g = cap;
    if (g < 1) g = 1;
    return (unsigned)g;
}
}  // namespace

// Inverse of node n's diagonal block: its dof row 4 n + i starts at
// 16 nrow_ptr[n] + 4 i deg, and the block is entries 4 diag_pos[n] .. + 3 of
// each row. Gauss-Jordan with partial pivoting in FP64; a zero pivot marks the
// node in *bad (the caller reports it).
template <typename T>
__global__ void k_bjac_invert(const T *vals, const int64_t *nrow_ptr, const int32_t *diag_pos,
                              int64_t n_nodes, double *dinv, int *bad) {
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= n_nodes) return;
    const int64_t b0 = nrow_ptr[n], deg = nrow_ptr[n + 1] - b0;
    const T *v = vals + 16 * b0 + 4 * (int64_t)diag_pos[n];
    double a[4][8];
    for (int i = 0; i < 4; ++i)
        for (int j = 0; j < 4; ++j) {
            a[i][j] = (double)v[4 * i * deg + j];
            a[i][4 + j] = i == j ? 1.0 : 0.0;
        }
    // partial pivoting by compare-and-swap against each lower row in turn (the
    // largest entry ends in the pivot row); fully unrolled so that every index
    // is static and the matrix stays in registers
#pragma unroll
    for (int c = 0; c < 4; ++c) {
#pragma unroll
        for (int r = c + 1; r < 4; ++r) {
            const bool sw = fabs(a[r][c]) > fabs(a[c][c]);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const double t = a[c][j];
                a[c][j] = sw ? a[r][j] : t;
                a[r][j] = sw ? t : a[r][j];
            }
        }
        if (a[c][c] == 0.0) {
            atomicOr(bad, 1);
            return;
        }
        const double ip = 1.0 / a[c][c];
#pragma unroll
        for (int j = 0; j < 8; ++j) a[c][j] *= ip;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (r == c) continue;
            const double f = a[r][c];
#pragma unroll
            for (int j = 0; j < 8; ++j) a[r][j] -= f * a[c][j];
        }
    }
    double *d = dinv + 16 * n;
    for (int i = 0; i < 4; ++i)
        for (int j = 0; j < 4; ++j) d[4 * i + j] = a[i][4 + j];
}

// entry i (0..3) of a diagonal block times x; d: its row
__device__ inline double block_row(const double *d, const double x[4]) {
    return __builtin_fma(d[3], x[3], __builtin_fma(d[2], x[2], __builtin_fma(d[0], x[0], d[1] * x[1])));
}
// the same by four lanes per node, one per entry (v: the lane's entry of x)
__device__ inline double block_row_lanes(const double *d, double v, int lane) {
    double x[4];
    for (int j = 0; j < 4; ++j) x[j] = __shfl(v, (lane & ~3) + j, 64);
    return block_row(d, x);
}
// y = blockdiag(dinv) x (a thread per entry: whole lines of dinv per wave)
__global__ void k_bjac_apply(const double *dinv, const double *x, double *y, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const double v = i < n ? x[i] : 0.0;
    const double *d = dinv + 4 * (i < n ? i : 0);
    const double r = block_row_lanes(d, v, threadIdx.x & 63);
    if (i < n) y[i] = r;
}

// Sums of a[0..3] over the wave, in a fixed order: lane l ends with that of
// a[l >> 4] (each exchange halves the values a lane keeps, then the lanes).
__device__ inline double wave_sum4(const double a[4], int lane) {
    const bool h = lane & 32, q = lane & 16;
    const double b0 = (h ? a[2] : a[0]) + __shfl_xor(h ? a[0] : a[2], 32, 64);
    const double b1 = (h ? a[3] : a[1]) + __shfl_xor(h ? a[1] : a[3], 32, 64);
    double c = (q ? b1 : b0) + __shfl_xor(q ? b0 : b1, 16, 64);
    for (int off = 8; off > 0; off >>= 1) c += __shfl_xor(c, off, 64);
    return c;
}

// One Gram-Schmidt sweep, a workgroup per chunk of KB entries of w (several
// chunks each on large systems). PROJ subtracts sum_k c[k] V_k from w first;
// then DOTS gives the chunk's share of V_k . w for every k < nk, without DOTS
// that of w . w. The subtraction and the next products share one read of V (the
// second from the caches). The loads' latency is the bound until the vectors
// outgrow the last-level cache: each wave has the loads of four k (products) or
// eight k (subtraction) in flight, and chunks are as small as a workgroup, so
// that short vectors still fill the chip. Partial sums: partial[k gridDim.x +
// block], fixed order.
constexpr int GS_MAXK = 201;
template <bool PROJ, bool DOTS>
__global__ __launch_bounds__(KB) void k_sweep(const double *V, int64_t ldv, int nk, const double *c, double *w,
                                              int64_t n, double *partial) {
    constexpr int NW = KB / 64;
    __shared__ double sw[KB];
    __shared__ double sc[PROJ ? GS_MAXK : 1];
    __shared__ double sacc[DOTS ? GS_MAXK : NW];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    if (PROJ)
        for (int k = t; k < nk; k += KB) sc[k] = c[k];
    if (DOTS)
        for (int k = t; k < nk; k += KB) sacc[k] = 0.0;
    double sq = 0.0;
    for (int64_t b = (int64_t)blockIdx.x * KB; b < n; b += (int64_t)gridDim.x * KB) {
        __syncthreads();
        const int64_t i = b + t;
        double v = i < n ? w[i] : 0.0;
        if (PROJ && i < n) {
            double s = 0.0;
#pragma unroll 8
            for (int k = 0; k < nk; ++k) s += sc[k] * V[(int64_t)k * ldv + i];
            v -= s;
            w[i] = v;
        }
        if (DOTS) {
            sw[t] = v;
            __syncthreads();
            for (int k0 = 4 * wv; k0 < nk; k0 += 4 * NW) {
                const double *Vk[4];
                for (int q = 0; q < 4; ++q) Vk[q] = V + (int64_t)(k0 + q < nk ? k0 + q : nk - 1) * ldv;
                double a[4] = {};
                if (b + KB <= n) {
                    double x[NW][4];
#pragma unroll
                    for (int u = 0; u < NW; ++u)
#pragma unroll
                        for (int q = 0; q < 4; ++q) x[u][q] = Vk[q][b + u * 64 + lane];
#pragma unroll
                    for (int u = 0; u < NW; ++u)
#pragma unroll
                        for (int q = 0; q < 4; ++q) a[q] += x[u][q] * sw[u * 64 + lane];
                } else {
                    for (int j = lane; b + j < n; j += 64)
                        for (int q = 0; q < 4; ++q) a[q] += Vk[q][b + j] * sw[j];
                }
                const double sum = wave_sum4(a, lane);
                const int k = k0 + (lane >> 4);
                if ((lane & 15) == 0 && k < nk) sacc[k] += sum;
            }
        } else {
            sq += v * v;
        }
    }
    if (DOTS) {
        __syncthreads();
        for (int k = t; k < nk; k += KB) partial[(int64_t)k * gridDim.x + blockIdx.x] = sacc[k];
    } else {
        for (int off = 32; off > 0; off >>= 1) sq += __shfl_down(sq, off, 64);
        if (lane == 0) sacc[wv] = sq;
        __syncthreads();
        if (t == 0) partial[blockIdx.x] = sacc[0] + sacc[1] + sacc[2] + sacc[3];
    }
}

// sum over the workgroup in a fixed order (thread 0 has it)
__device__ inline double block_sum(double v, double *sh) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    return sh[0] + sh[1] + sh[2] + sh[3];
}

// partial[k gridDim.x + block]: the block's share of V_k . w for k < NK
template <int NK>
__global__ __launch_bounds__(KB) void k_dots(const double *V, int64_t ldv, const double *w, int64_t n,
                                             double *partial) {
    __shared__ double red[4];
    double a[NK] = {};
    for (int64_t i = (int64_t)blockIdx.x * KB + threadIdx.x; i < n; i += (int64_t)gridDim.x * KB) {
        const double x = w[i];
        for (int k = 0; k < NK; ++k) a[k] += V[(int64_t)k * ldv + i] * x;
    }
    for (int k = 0; k < NK; ++k) {
        const double s = block_sum(a[k], red);
        if (threadIdx.x == 0) partial[(int64_t)k * gridDim.x + blockIdx.x] = s;
    }
}

// out[k] = sum of the nb partial sums of row k, in a fixed order (a wave per k,
// the loads of up to 1024 sums in flight at once); host (nullable, host memory the
// device can write): a copy of the sums and of the `before` entries ahead of out
__global__ __launch_bounds__(64) void k_sums(const double *partial, int nb, double *out, double *host, int before) {
    const int k = blockIdx.x, l = threadIdx.x;
    double v[16], s = 0.0;
#pragma unroll
    for (int q = 0; q < 16; ++q) v[q] = l + 64 * q < nb ? partial[(int64_t)k * nb + l + 64 * q] : 0.0;
#pragma unroll
    for (int q = 0; q < 16; ++q) s += v[q];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
    if (l == 0) {
        out[k] = s;
        if (host) host[before + k] = s;
    }
    if (host && k == 0)
        for (int i = l; i < before; i += 64) host[i] = out[i - before];
}

// v = w / sqrt(*norm2), z = blockdiag(dinv) v
__global__ void k_next_vector(const double *w, const double *norm2, const double *dinv, double *v, double *z,
                              int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const double a = i < n ? (1.0 / sqrt(*norm2)) * w[i] : 0.0;
    const double y = block_row_lanes(dinv + 4 * (i < n ? i : 0), a, threadIdx.x & 63);
    if (i < n) {
        v[i] = a;
        z[i] = y;
    }
}

// ---- BiCGStab: vector updates with their preconditioner and inner products ----
//
// The recurrence amplifies rounding errors (1e-16 in one sum is 1e-9 in the
// solution after 15 steps on some meshes), so the order of the sums and the
// places of the fused multiply-adds are spelled out.
__device__ inline double add_unfused(double a, double b, double c) {  // a + b c, product rounded
#pragma clang fp contract(off)
    const double m = b * c;
    return a + m;
}

// p = r (first) or r + beta (p - omega v); ph = blockdiag(dinv) p
__global__ void k_bcgs_p(int first, double beta, double omega, const double *r, const double *v, const double *dinv,
                         double *p, double *ph, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double a = 0.0;
    if (i < n) p[i] = a = first ? r[i] : __builtin_fma(-beta * omega, v[i], add_unfused(r[i], beta, p[i]));
    const double y = block_row_lanes(dinv + 4 * (i < n ? i : 0), a, threadIdx.x & 63);
    if (i < n) ph[i] = y;
}

// alpha = rho / (rh . v), 0 if that vanishes (dot: device)
__device__ inline double bcgs_alpha(double rho, const double *dot) { return dot[0] != 0.0 ? rho / dot[0] : 0.0; }

// s = r - alpha v, sh = blockdiag(dinv) s; partial: shares of s . s
__global__ __launch_bounds__(KB) void k_bcgs_s(double rho, const double *dot, const double *r, const double *v,
                                               const double *dinv, double *s, double *sh, int64_t n,
                                               double *partial) {
    __shared__ double red[4];
    const double alpha = bcgs_alpha(rho, dot);
    double sq = 0.0;
    for (int64_t b = (int64_t)blockIdx.x * KB; b < n; b += (int64_t)gridDim.x * KB) {
        const int64_t i = b + threadIdx.x;
        const double a = i < n ? add_unfused(r[i], -alpha, v[i]) : 0.0;
        const double y = block_row_lanes(dinv + 4 * (i < n ? i : 0), a, threadIdx.x & 63);
        if (i < n) {
            s[i] = a;
            sh[i] = y;
        }
        sq += a * a;
    }
    const double all = block_sum(sq, red);
    if (threadIdx.x == 0) partial[blockIdx.x] = all;
}

// omega = (s . t) / (t . t), 0 where the step ends at x + alpha ph (rh . v = 0,
// |s| <= tol, t = 0); x += alpha ph + omega sh, r = s - omega t; partial:
// shares of r . r and rh . r. dots (device): rh . v, s . s, s . t, t . t
__global__ __launch_bounds__(KB) void k_bcgs_x(double rho, double tol, const double *dots, const double *ph,
                                               const double *sh, const double *s, const double *t, const double *rh,
                                               double *x, double *r, int64_t n, double *partial) {
    __shared__ double red[4];
    if (dots[0] == 0.0) return;  // the caller stops without a step
    const double alpha = bcgs_alpha(rho, dots);
    const bool end = sqrt(dots[1]) <= tol || dots[3] == 0.0;
    const double omega = end ? 0.0 : dots[2] / dots[3];
    double rr = 0.0, rhr = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * KB + threadIdx.x; i < n; i += (int64_t)gridDim.x * KB) {
        const double half = add_unfused(x[i], alpha, ph[i]);
        x[i] = end ? half : __builtin_fma(omega, sh[i], half);
        const double v = end ? s[i] : add_unfused(s[i], -omega, t[i]);
        r[i] = v;
        rr += v * v;
        rhr += rh[i] * v;
    }
    rr = block_sum(rr, red);
    rhr = block_sum(rhr, red);
    if (threadIdx.x == 0) {
        partial[blockIdx.x] = rr;
        partial[gridDim.x + blockIdx.x] = rhr;
    }
}

// w = sum_k c[k] V_k (c on the device)
__global__ void k_combine(const double *V, int64_t ldv, int nk, const double *c, double *w, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * KB + threadIdx.x; i < n; i += (int64_t)gridDim.x * KB) {
        double s = 0.0;
        for (int k = 0; k < nk; ++k) s += c[k] * V[(int64_t)k * ldv + i];
        w[i] = s;
    }
}

// out = a x + b y (host scalars; out may alias x or y)
__global__ void k_axpby(double a, const double *x, double b, const double *y, double *out, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * KB + threadIdx.x; i < n; i += (int64_t)gridDim.x * KB)
        out[i] = a * x[i] + b * y[i];
}

void launch_bjac_invert_f64(hipStream_t s, const double *vals, const int64_t *nrow_ptr,
                            const int32_t *diag_pos, int64_t n_nodes, double *dinv, int *bad) {
    if (n_nodes > 0)
        hipLaunchKernelGGL(k_bjac_invert<double>, dim3((unsigned)((n_nodes + 127) / 128)), dim3(128), 0, s,
                           vals, nrow_ptr, diag_pos, n_nodes, dinv, bad);
}
void launch_bjac_invert_f32(hipStream_t s, const float *vals, const int64_t *nrow_ptr,
                            const int32_t *diag_pos, int64_t n_nodes, double *dinv, int *bad) {
    if (n_nodes > 0)
        hipLaunchKernelGGL(k_bjac_invert<float>, dim3((unsigned)((n_nodes + 127) / 128)), dim3(128), 0, s,
                           vals, nrow_ptr, diag_pos, n_nodes, dinv, bad);
}
void launch_bjac_apply(hipStream_t s, const double *dinv, const double *x, double *y, int64_t n_nodes) {
    if (n_nodes > 0)
        hipLaunchKernelGGL(k_bjac_apply, dim3((unsigned)((4 * n_nodes + KB - 1) / KB)), dim3(KB), 0, s, dinv, x, y,
                           4 * n_nodes);
}
int sweep_blocks(int64_t n) { return (int)blocks_for(n, 1024); }
void launch_sweep(hipStream_t s, const double *V, int64_t ldv, int nk, const double *c, bool dots, double *w, int64_t n,
                  double *partial, double *out, double *host, int before) {
    const unsigned nb = (unsigned)sweep_blocks(n);
    if (c && dots) hipLaunchKernelGGL((k_sweep<true, true>), dim3(nb), dim3(KB), 0, s, V, ldv, nk, c, w, n, partial);
    else if (c) hipLaunchKernelGGL((k_sweep<true, false>), dim3(nb), dim3(KB), 0, s, V, ldv, nk, c, w, n, partial);
    else if (nk > 0) hipLaunchKernelGGL((k_sweep<false, true>), dim3(nb), dim3(KB), 0, s, V, ldv, nk, c, w, n, partial);
    hipLaunchKernelGGL(k_sums, dim3(dots ? (unsigned)nk : 1u), dim3(64), 0, s, partial, (int)nb, out, host, before);
}
void launch_dots(hipStream_t s, const double *V, int64_t ldv, int nk, const double *w, int64_t n, double *partial,
                 double *out, double *host, int before) {
    const unsigned nb = blocks_for(n, 1024);
    if (nk == 1) hipLaunchKernelGGL(k_dots<1>, dim3(nb), dim3(KB), 0, s, V, ldv, w, n, partial);
    else hipLaunchKernelGGL(k_dots<2>, dim3(nb), dim3(KB), 0, s, V, ldv, w, n, partial);
    hipLaunchKernelGGL(k_sums, dim3((unsigned)nk), dim3(64), 0, s, partial, (int)nb, out, host, before);
}
void launch_next_vector(hipStream_t s, const double *w, const double *norm2, const double *dinv, double *v, double *z,
                        int64_t n_nodes) {
    if (n_nodes > 0)
        hipLaunchKernelGGL(k_next_vector, dim3((unsigned)((4 * n_nodes + KB - 1) / KB)), dim3(KB), 0, s, w, norm2, dinv,
                           v, z, 4 * n_nodes);
}
void launch_bcgs_p(hipStream_t s, bool first, double beta, double omega, const double *r, const double *v,
                   const double *dinv, double *p, double *ph, int64_t n_nodes) {
    if (n_nodes > 0)
        hipLaunchKernelGGL(k_bcgs_p, dim3((unsigned)((4 * n_nodes + KB - 1) / KB)), dim3(KB), 0, s, first ? 1 : 0, beta,
                           omega, r, v, dinv, p, ph, 4 * n_nodes);
}
void launch_bcgs_s(hipStream_t s, double rho, const double *dot, const double *r, const double *v, const double *dinv,
                   double *sv, double *sh, int64_t n_nodes, double *partial, double *out) {
    const unsigned nb = blocks_for(4 * n_nodes, 1024);
    hipLaunchKernelGGL(k_bcgs_s, dim3(nb), dim3(KB), 0, s, rho, dot, r, v, dinv, sv, sh, 4 * n_nodes, partial);
    hipLaunchKernelGGL(k_sums, dim3(1), dim3(64), 0, s, partial, (int)nb, out, nullptr, 0);
}
void launch_bcgs_x(hipStream_t s, double rho, double tol, const double *dots, const double *ph, const double *sh,
                   const double *sv, const double *t, const double *rh, double *x, double *r, int64_t n,
                   double *partial, double *out, double *host, int before) {
    const unsigned nb = blocks_for(n, 1024);
    hipLaunchKernelGGL(k_bcgs_x, dim3(nb), dim3(KB), 0, s, rho, tol, dots, ph, sh, sv, t, rh, x, r, n, partial);
    hipLaunchKernelGGL(k_sums, dim3(2), dim3(64), 0, s, partial, (int)nb, out, host, before);
}
void launch_combine(hipStream_t s, const double *V, int64_t ldv, int nk, const double *c, double *w, int64_t n) {
    if (n > 0) hipLaunchKernelGGL(k_combine, dim3(blocks_for(n, 4096)), dim3(KB), 0, s, V, ldv, nk, c, w, n);
}
void launch_axpby(hipStream_t s, double a, const double *x, double b, const double *y, double *out,
                  int64_t n) {
    if (n > 0)
        hipLaunchKernelGGL(k_axpby, dim3(blocks_for(n, 4096)), dim3(KB), 0, s, a, x, b, y, out, n);
}

}  // namespace vmsk
