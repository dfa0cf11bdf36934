// measure.hip -- measurements on a gauge configuration at the end of a
// trajectory (Sec. 3: after each trajectory the program measures on the
// configuration; the observables are not named there).  Built here: the
// Polyakov loop and the point-source propagator with the pion correlator;
// the plaquette comes with the HMC code.
//
// Propagator: column j = 3*spin + colour solves M psi_j = b_j, b_j a unit
// point source at `src`.  With M = [[1, -k D_eo], [-k D_oe, 1]] in even-odd
// blocks,
//   Mhat psi_e = b_e + k D_eo b_o,   psi_o = b_o + k D_oe psi_e,
// and Mhat psi_e = bhat is solved as Mhat^dag Mhat psi_e = Mhat^dag bhat by the
// batched CG (all 12 columns in one multi-RHS solve, any sloppy precision),
// Mhat^dag = 1 - k^2 D_oe^dag D_eo^dag.  Sums are FP64 in a fixed order.
#include <stdio.h>

#include <cmath>
#include <cstring>
#include <vector>

#include "m3.h"
#include "wd_internal.h"

namespace wd {

namespace {

constexpr int kB = 256;

#define HIPCHK(expr)                                                                               \
    do {                                                                                          \
        hipError_t e__ = (expr);                                                                  \
        if (e__ != hipSuccess)                                                                    \
            return set_error(WD_ERR_HIP, "%s: %s (%s:%d)", #expr, hipGetErrorString(e__), __FILE__, __LINE__); \
    } while (0)

inline unsigned nblk(long long n) { return (unsigned)((n + kB - 1) / kB); }

__global__ void __launch_bounds__(kB) k_fill(double *a, double v, long long n)
{
    const long long i = (long long)blockIdx.x * kB + threadIdx.x;
    if (i < n) a[i] = v;
}

// column j of a [12][sites][4][3] field gets +1 at (site, spin-colour j)
__global__ void k_add_point(double *b, int site, long long col_doubles)
{
    const int j = threadIdx.x;
    if (j < 12) b[(size_t)j * col_doubles + (size_t)site * 24 + 2 * j] += 1.0;
}

// Fixed-order block sum of kB values (tree over shared memory).
__device__ inline double block_sum(double v, double *sh)
{
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int off = kB / 2; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) sh[threadIdx.x] += sh[threadIdx.x + off];
        __syncthreads();
    }
    return sh[0];
}

// partial[t * nb + b] = sum over the spatial sites [b*kB, (b+1)*kB) of time
// slice t of |psi_j|^2, all 12 columns and 12 spin-colour entries.
__global__ void __launch_bounds__(kB) k_corr_partial(const double *psi, long long V, int v3, int nb,
                                                     double *partial)
{
    __shared__ double sh[kB];
    const int b = blockIdx.x, t = blockIdx.y;
    const int s = b * kB + threadIdx.x;
    double acc = 0.0;
    if (s < v3) {
        const size_t site = (size_t)t * v3 + s;
        for (int j = 0; j < 12; j++) {
            const double *p = psi + ((size_t)j * V + site) * 24;
#pragma unroll
            for (int k = 0; k < 24; k++) acc = fmaT(p[k], p[k], acc);
        }
    }
    const double tot = block_sum(acc, sh);
    if (threadIdx.x == 0) partial[(size_t)t * nb + b] = tot;
}

// out[dt] = sum_b partial[((t0 + dt) mod Lt) * nb + b], in b order
__global__ void k_corr_final(const double *partial, int nb, int Lt, int t0, double *out)
{
    const int dt = blockIdx.x * blockDim.x + threadIdx.x;
    if (dt >= Lt) return;
    const int t = (t0 + dt) % Lt;
    double s = 0.0;
    for (int b = 0; b < nb; b++) s += partial[(size_t)t * nb + b];
    out[dt] = s;
}

// Per spatial site s: (1/3) tr prod_{t = 0..Lt-1} U_t(s, t).  A work-group
// takes kRowLinks sites, three lanes a site; each of its kPolySeg waves
// multiplies the links of a contiguous range of t, and the first wave
// multiplies the ranges in order.  partial[2 * b + {0, 1}]: (Re, Im) summed
// over the sites.  A chain of Lt dependent products per thread over v3 threads
// left most of the chip idle: 24^3 x 48 101 us, 28 now.
constexpr int kPolySeg = 8;
__global__ void __launch_bounds__(64 * kPolySeg) k_poly_partial(const double *U, int v3, int Lt, double *partial)
{
    __shared__ dbl2_t sh[kPolySeg][kRowWords];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, row = lane % 3;
    dbl2_t *lds = sh[w];
    const int s0 = blockIdx.x * kRowLinks + lane / 3;
    const int s = s0 < v3 ? s0 : v3 - 1;
    Row3 P;
#pragma unroll
    for (int k = 0; k < 3; k++) P.e[k] = make_double2(k == row ? 1.0 : 0.0, 0.0);
    const int t1 = Lt * (w + 1) / kPolySeg;
#pragma unroll 1
    for (int t = Lt * w / kPolySeg; t < t1; t += 3) {
        // three links in flight; those past the range are fetched but not used
        const LinkWords f0 = fetch_links(U, (t * v3 + s) * 4 + 3),
                        f1 = fetch_links(U, ((t + 1 < t1 ? t + 1 : t) * v3 + s) * 4 + 3),
                        f2 = fetch_links(U, ((t + 2 < t1 ? t + 2 : t) * v3 + s) * 4 + 3);
        stage_links(f0, lds);
        P = row_mul(P, lds);
        if (t + 1 < t1) {
            stage_links(f1, lds);
            P = row_mul(P, lds);
        }
        if (t + 2 < t1) {
            stage_links(f2, lds);
            P = row_mul(P, lds);
        }
    }
    __syncthreads();  // (all lanes are done with the staged links)
#pragma unroll
    for (int k = 0; k < 3; k++) lds[lane * 3 + k] = dbl2_t{P.e[k].x, P.e[k].y};
    __syncthreads();
    if (w != 0) return;
    for (int q = 1; q < kPolySeg; q++) P = row_mul(P, sh[q]);
    const bool live = lane < 3 * kRowLinks && s0 < v3;
    double re = row == 0 ? P.e[0].x : (row == 1 ? P.e[1].x : P.e[2].x);
    double im = row == 0 ? P.e[0].y : (row == 1 ? P.e[1].y : P.e[2].y);
    re = live ? re / 3.0 : 0.0;
    im = live ? im / 3.0 : 0.0;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        re += __shfl_xor(re, off, 64);
        im += __shfl_xor(im, off, 64);
    }
    if (lane == 0) {
        partial[2 * blockIdx.x] = re;
        partial[2 * blockIdx.x + 1] = im;
    }
}

// out = sum over the nb partials / v3, each lane of one wave every 64th, then
// a fixed tree
__global__ void __launch_bounds__(64) k_poly_final(const double *partial, int nb, int v3, double *out)
{
    double re = 0.0, im = 0.0;
    for (int b = threadIdx.x; b < nb; b += 64) {
        re += partial[2 * b];
        im += partial[2 * b + 1];
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        re += __shfl_xor(re, off, 64);
        im += __shfl_xor(im, off, 64);
    }
    if (threadIdx.x == 0) {
        out[0] = re / v3;
        out[1] = im / v3;
    }
}

wd_status check_src(const wd_ctx *c, const int32_t src[4])
{
    if (!src) return set_error(WD_ERR_ARG, "NULL source");
    for (int mu = 0; mu < 4; mu++)
        if (src[mu] < 0 || src[mu] >= c->dims[mu])
            return set_error(WD_ERR_ARG, "source coordinate %d = %d outside 0..%d", mu, src[mu], c->dims[mu] - 1);
    return WD_OK;
}

wd_status read_back(wd_ctx *c, double *host, const double *dev, int n)
{
    void *h;
    WD_TRY(pinned_get(c, 1, sizeof(double) * n, &h));
    HIPCHK(hipMemcpyAsync(h, dev, sizeof(double) * n, hipMemcpyDeviceToHost, c->stream));
    HIPCHK(hipStreamSynchronize(c->stream));
    std::memcpy(host, h, sizeof(double) * n);
    return WD_OK;
}

}  // namespace

}  // namespace wd

using namespace wd;

extern "C" wd_status wd_polyakov(wd_ctx *c, const double *U, double *out)
{
    if (!c || !U || !out) return set_error(WD_ERR_ARG, "NULL argument");
    WD_HIP(hipSetDevice(c->device));
    const int v3 = c->dims[0] * c->dims[1] * c->dims[2], Lt = c->dims[3];
    const int nb = (v3 + kRowLinks - 1) / kRowLinks;
    void *vp;
    WD_TRY(ws_get(c, "ms_poly", sizeof(double) * (2 * nb + 2), &vp));
    double *partial = (double *)vp, *res = partial + 2 * nb;
    hipLaunchKernelGGL(k_poly_partial, dim3(nb), dim3(64 * kPolySeg), 0, c->stream, U, v3, Lt, partial);
    hipLaunchKernelGGL(k_poly_final, dim3(1), dim3(64), 0, c->stream, partial, nb, v3, res);
    HIPCHK(hipGetLastError());
    return read_back(c, out, res, 2);
}

extern "C" wd_status wd_point_propagator(wd_ctx *c, double *psi, const int32_t src[4], double kappa,
                                         const wd_solver_params *pin, wd_solver_stats *st)
{
    if (!c || !psi) return set_error(WD_ERR_ARG, "NULL argument");
    if (!c->have_gauge) return set_error(WD_ERR_STATE, "no gauge field loaded");
    WD_TRY(check_src(c, src));
    if (!std::isfinite(kappa)) return set_error(WD_ERR_ARG, "kappa not finite");
    wd_solver_params p;
    wd_solver_defaults(&p);
    if (pin) p = *pin;
    if (!p.eo) return set_error(WD_ERR_ARG, "the propagator uses the even-odd solve (eo = 1)");
    WD_HIP(hipSetDevice(c->device));
    const hipStream_t s = c->stream;
    const long long col = c->Vh * 24;  // doubles per parity column
    const int x0 = src[0] + c->dims[0] * (src[1] + c->dims[1] * (src[2] + c->dims[2] * src[3]));
    const int par = (src[0] + src[1] + src[2] + src[3]) & 1, cb0 = x0 >> 1;
    void *vp;
    WD_TRY(ws_get(c, "ms_a", sizeof(double) * 12 * col, &vp));
    double *A = (double *)vp;  // bhat, then the even solution
    WD_TRY(ws_get(c, "ms_b", sizeof(double) * 12 * col, &vp));
    double *B = (double *)vp;  // Mhat^dag bhat
    // (the twelve columns of a step in one launch; psi, written last, holds
    // intermediate parity columns: from here on no argument is refused and no
    // memory is asked for)
    WD_TRY(cg_prepare(c, 12, p));
    // bhat_j = b_e + k D_eo b_o
    hipLaunchKernelGGL(k_fill, dim3(nblk(12 * col)), dim3(kB), 0, s, A, 0.0, 12 * col);
    if (par == 0) {
        hipLaunchKernelGGL(k_add_point, dim3(1), dim3(64), 0, s, A, cb0, col);
    } else {
        hipLaunchKernelGGL(k_fill, dim3(nblk(12 * col)), dim3(kB), 0, s, psi, 0.0, 12 * col);
        hipLaunchKernelGGL(k_add_point, dim3(1), dim3(64), 0, s, psi, cb0, col);
        OpArgs o;
        o.incanon = o.xpay = o.xcanon = o.outcanon = 1;
        o.in = (const char *)psi;
        o.coef = kappa;
        o.x = (const char *)A;
        o.out = (char *)A;
        o.in_rs = o.x_rs = o.out_rs = col;
        WD_TRY(op_sweep(c, o, SP_F64, c->lk64, 0, 12));
    }
    HIPCHK(hipGetLastError());
    // B_j = Mhat^dag bhat_j
    WD_TRY(mhat_dag_apply(c, B, A, psi, kappa, 12));
    // psi_e: the batched solve of all 12 columns
    std::vector<double> kap(12, kappa);
    const wd_status sst = wd_cg_solve(c, A, B, 12, kap.data(), &p, st);
    if (sst != WD_OK && sst != WD_ERR_NOCONV && sst != WD_ERR_NAN) return sst;
    // psi_o = b_o + k D_oe psi_e, merged with psi_e into the full columns
    OpArgs o;
    o.P0 = 1;
    o.incanon = o.outcanon = 1;
    o.in = (const char *)A;
    o.out = (char *)B;
    o.in_rs = o.out_rs = col;
    WD_TRY(op_sweep(c, o, SP_F64, c->lk64, 0, 12));
    HIPCHK(merge_parities(A, B, kappa, psi, 12, c->g, s));
    if (par == 1) hipLaunchKernelGGL(k_add_point, dim3(1), dim3(64), 0, s, psi, x0, 2 * col);
    HIPCHK(hipGetLastError());
    HIPCHK(hipStreamSynchronize(s));
    if (sst != WD_OK) set_error(sst, "%s", sst == WD_ERR_NAN ? "non-finite residual" : "not converged");
    return sst;
}

extern "C" wd_status wd_pion_correlator(wd_ctx *c, double *corr, const double *psi, const int32_t src[4])
{
    if (!c || !corr || !psi) return set_error(WD_ERR_ARG, "NULL argument");
    WD_TRY(check_src(c, src));
    WD_HIP(hipSetDevice(c->device));
    const int v3 = c->dims[0] * c->dims[1] * c->dims[2], Lt = c->dims[3];
    const int nb = (int)nblk(v3);
    void *vp;
    WD_TRY(ws_get(c, "ms_corr", sizeof(double) * ((size_t)nb * Lt + Lt), &vp));
    double *partial = (double *)vp, *res = partial + (size_t)nb * Lt;
    hipLaunchKernelGGL(k_corr_partial, dim3(nb, Lt), dim3(kB), 0, c->stream, psi, (long long)2 * c->Vh, v3, nb,
                       partial);
    hipLaunchKernelGGL(k_corr_final, dim3((Lt + 63) / 64), dim3(64), 0, c->stream, partial, nb, Lt, src[3], res);
    HIPCHK(hipGetLastError());
    return read_back(c, corr, res, Lt);
}
