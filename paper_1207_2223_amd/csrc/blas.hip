// blas.hip -- CG vector kernels over batches of spinor fields (the level-1
// BLAS work the paper delegates to CUBLAS, Sec. 3), fused where CG allows,
// with deterministic FP64 reductions: each group of 16 consecutive sites
// writes one partial sum in a fixed pairing order, and blas_finalize adds the
// partials of one RHS in a fixed order in a single work-group.
#include "wd_internal.h"

namespace wd {

namespace {

constexpr int kBlock = 256;

// fin_wave_sum's value (the order of every CG scalar's sum) by a work-group of
// kBlock threads: thread t sums the virtual lanes t + kBlock q, pairs them as
// the halving tree does, ((q0 + q2) + (q1 + q3)), and the rest of the tree
// pairs threads: two levels over LDS, six within the first wave.  The result
// is in every thread; sh: kBlock doubles, free again after the call's last
// barrier.  (One thread a virtual lane, a barrier a level: 4.4 us for the 4096
// partials of 16^3 x 32 with one RHS, 3.2 now.)
__device__ __forceinline__ double fin_block_sum(const double *pp, int nw, double *sh)
{
    static_assert(kFinLanes == 4 * kBlock, "four virtual lanes a thread");
    const int t = (int)threadIdx.x;
    double q[4] = {0.0, 0.0, 0.0, 0.0};
    for (int w0 = 0; w0 < nw; w0 += 4 * kFinLanes) {
        double x[4][4];
#pragma unroll
        for (int m = 0; m < 4; m++)
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const int w = w0 + t + kBlock * i + m * kFinLanes;
                x[i][m] = w < nw ? pp[w] : 0.0;
            }
#pragma unroll
        for (int i = 0; i < 4; i++)
#pragma unroll
            for (int m = 0; m < 4; m++) q[i] += x[i][m];
    }
    sh[t] = (q[0] + q[2]) + (q[1] + q[3]);
    __syncthreads();
    if (t < 64) {
        double v = (sh[t] + sh[t + 128]) + (sh[t + 64] + sh[t + 192]);
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            const double o = __shfl_down(v, off, 64);
            if (t < off) v += o;
        }
        if (t == 0) sh[0] = v;
    }
    __syncthreads();
    return sh[0];
}

__device__ __forceinline__ double sum16(double v)
{
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

struct FArg {
    char *base;
    long long rs, ss;
    int cs;
};
inline FArg fa(const Field &f) { return FArg{f.base, f.rs, f.ss, f.cs}; }

__device__ __forceinline__ char *site_base(const FArg &f, int rid, int sub)
{
    return f.base + rid * f.rs + sub * f.ss;
}

template <int SP>
__global__ void __launch_bounds__(kBlock) k_norm(FArg a, int Vh, int nsub, const int *active,
                                                  double *partial, int pstride)
{
    typedef typename SpinorIO<SP>::real real;
    const int rid = active[blockIdx.y];
    const int s = blockIdx.x * kBlock + threadIdx.x;
    double v = 0.0;
    if (s < nsub * Vh) {
        const int sub = s / Vh, i = s - sub * Vh;
        real x[24];
        SpinorIO<SP>::load(site_base(a, rid, sub), a.cs, i, x);
#pragma unroll
        for (int k = 0; k < 24; k++) v = fmaT((double)x[k], (double)x[k], v);
    }
    v = sum16(v);
    if ((threadIdx.x & 15) == 0 && s < nsub * Vh) partial[(size_t)rid * pstride + (s >> 4)] = v;
}

template <int SP>
__global__ void __launch_bounds__(kBlock) k_p_update(FArg p, FArg r, const double *beta, int Vh,
                                                      int nsub, const int *active)
{
    typedef typename SpinorIO<SP>::real real;
    const int rid = active[blockIdx.y];
    const int s = blockIdx.x * kBlock + threadIdx.x;
    if (s >= nsub * Vh) return;
    const int sub = s / Vh, i = s - sub * Vh;
    const real b = (real)beta[rid];
    real pv[24], rv[24];
    SpinorIO<SP>::load(site_base(p, rid, sub), p.cs, i, pv);
    SpinorIO<SP>::load(site_base(r, rid, sub), r.cs, i, rv);
#pragma unroll
    for (int k = 0; k < 24; k++) pv[k] = fmaT(b, pv[k], rv[k]);
    SpinorIO<SP>::store(site_base(p, rid, sub), p.cs, i, pv);
}

// The directions p[0..m-1] of the last m iterations (ring slots, RHS stride rs).
struct Ring {
    const char *base[kMaxRing];
    long long rs;
};

// beta of an iteration, finalized by every work-group of the p update for
// itself: beta = (sum of the nw partials) / rr_in, written with the sum to
// beta and rr_out by the first work-group of a RHS (rr_in and rr_out differ,
// so that no other reads what it writes).  partial == nullptr: beta is read.
struct BetaArg {
    const double *partial;
    int pstride, nw;
    const double *rr_in;
    double *rr_out, *beta, *hout;
};

// pd = r + beta p[m-1]; with FLUSH first x += alpha_j p[j] for j = 0..m-1,
// in that order (the order and roundings of advancing x once per iteration).
// Bound by memory; p and r are loaded before the sum for beta is waited for.
// The sum saves a launch an iteration (finalize and its gap, 4-6 us) and costs
// each work-group nw doubles from the L2: 8^3 x 16 3.0 -> 3.8 us, 16^3 x 32 5.4
// -> 6.4.
template <int SP, int XP, bool FLUSH>
__global__ void __launch_bounds__(kBlock) k_p_update_ring(Ring p, int m, FArg pd, FArg r, BetaArg bt,
                                                           FArg x, const double *ahist, int ahs, int Vh,
                                                           const int *active)
{
    typedef typename SpinorIO<SP>::real real;
    typedef typename SpinorIO<XP>::real xreal;
    __shared__ double sh[kBlock];
    const int rid = active[blockIdx.y];
    const int i = blockIdx.x * kBlock + threadIdx.x;
    const bool live = i < Vh;
    const int is = live ? i : Vh - 1;
    real pv[24], rv[24];
    if constexpr (FLUSH) {
        if (live) {
            xreal xv[24];
            SpinorIO<XP>::load(x.base + rid * x.rs, x.cs, i, xv);
#pragma unroll
            for (int j = 0; j < kMaxRing; j++) {
                if (j < m) {
                    const real al = (real)ahist[(size_t)j * ahs + rid];
                    SpinorIO<SP>::load(p.base[j] + rid * p.rs, pd.cs, i, pv);
#pragma unroll
                    for (int k = 0; k < 24; k++) xv[k] = fmaT((xreal)al, (xreal)pv[k], xv[k]);
                }
            }
            SpinorIO<XP>::store(x.base + rid * x.rs, x.cs, i, xv);
        }
    } else {
        SpinorIO<SP>::load(p.base[m - 1] + rid * p.rs, pd.cs, is, pv);
    }
    SpinorIO<SP>::load(r.base + rid * r.rs, r.cs, is, rv);
    real b;
    if (bt.partial) {
        const double s = fin_block_sum(bt.partial + (size_t)rid * bt.pstride, bt.nw, sh), bd = s / bt.rr_in[rid];
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            bt.rr_out[rid] = s;
            bt.beta[rid] = bd;
            if (bt.hout) {
                bt.hout[rid] = s;
                __threadfence_system();
            }
        }
        b = (real)bd;
    } else {
        b = (real)bt.beta[rid];
    }
    if (!live) return;
#pragma unroll
    for (int k = 0; k < 24; k++) pv[k] = fmaT(b, pv[k], rv[k]);
    SpinorIO<SP>::store(pd.base + rid * pd.rs, pd.cs, i, pv);
}

template <int SP, int XP>
__global__ void __launch_bounds__(kBlock) k_cg_update(FArg x, FArg p, FArg r, FArg Ap,
                                                       const double *alpha, int Vh, int nsub,
                                                       const int *active, double *partial,
                                                       int pstride)
{
    typedef typename SpinorIO<SP>::real real;
    typedef typename SpinorIO<XP>::real xreal;
    const int rid = active[blockIdx.y];
    const int s = blockIdx.x * kBlock + threadIdx.x;
    double v = 0.0;
    if (s < nsub * Vh) {
        const int sub = s / Vh, i = s - sub * Vh;
        const real al = (real)alpha[rid];
        real pv[24], rv[24], av[24];
        xreal xv[24];
        SpinorIO<SP>::load(site_base(p, rid, sub), p.cs, i, pv);
        SpinorIO<SP>::load(site_base(r, rid, sub), r.cs, i, rv);
        SpinorIO<SP>::load(site_base(Ap, rid, sub), Ap.cs, i, av);
        SpinorIO<XP>::load(site_base(x, rid, sub), x.cs, i, xv);
#pragma unroll
        for (int k = 0; k < 24; k++) {
            xv[k] = fmaT((xreal)al, (xreal)pv[k], xv[k]);
            rv[k] = fmaT(-al, av[k], rv[k]);
            v = fmaT((double)rv[k], (double)rv[k], v);
        }
        SpinorIO<XP>::store(site_base(x, rid, sub), x.cs, i, xv);
        SpinorIO<SP>::store(site_base(r, rid, sub), r.cs, i, rv);
    }
    v = sum16(v);
    if ((threadIdx.x & 15) == 0 && s < nsub * Vh) partial[(size_t)rid * pstride + (s >> 4)] = v;
}

template <int SP>
__global__ void __launch_bounds__(kBlock) k_copy(FArg d, FArg src, int Vh, int nsub, const int *active)
{
    const int rid = active[blockIdx.y];
    const int s = blockIdx.x * kBlock + threadIdx.x;
    if (s >= nsub * Vh) return;
    const int sub = s / Vh, i = s - sub * Vh;
    double v[24];
    SpinorIO<SP>::load(site_base(src, rid, sub), src.cs, i, v);
    SpinorIO<SP>::store(site_base(d, rid, sub), d.cs, i, v);
}

// Store of 24 reals and what a load of them gives back.
template <int SP, typename T>
__device__ __forceinline__ void store_rt(char *f, int cs, int i, const T v[24], typename SpinorIO<SP>::real back[24])
{
    if constexpr (has_norm(SP)) {
        uint32_t w[12];
        const float n = SpinorIO<SP>::encode(v, w);
        u32x4_t *p = reinterpret_cast<u32x4_t *>(f);
#pragma unroll
        for (int k = 0; k < 3; k++) p[(size_t)k * cs + i] = u32x4_t{w[4 * k], w[4 * k + 1], w[4 * k + 2], w[4 * k + 3]};
        reinterpret_cast<float *>(f + (size_t)48 * cs)[i] = n;
#pragma unroll
        for (int k = 0; k < 12; k++) SpinorIO<SP>::decode(w[k], n, &back[2 * k], &back[2 * k + 1]);
    } else {
#pragma unroll
        for (int k = 0; k < 24; k++) back[k] = (typename SpinorIO<SP>::real)v[k];
        SpinorIO<SP>::store(f, cs, i, back);
    }
}

struct IdList {
    int n;
    int id[64];
};
__global__ void k_set_ids(int *dst, IdList l)
{
    if ((int)threadIdx.x < l.n) dst[threadIdx.x] = l.id[threadIdx.x];
}

struct CoefList {
    int n;
    int id[32];
    double kappa[32];
};
__global__ void k_set_coefs(double *c1, double *c2, CoefList l)
{
    const int q = threadIdx.x;
    if (q >= l.n) return;
    const double k = l.kappa[q];
    c1[l.id[q]] = -k;
    c2[l.id[q]] = -k * k;
}

// (see blas_cg_init) One pass over the fields of a new right-hand side; as
// separate norm, zero and copy launches it was seven.
template <int SP, bool FRESH>
__global__ void __launch_bounds__(kBlock) k_cg_init(FArg b, FArg x, FArg r, FArg rs, FArg xs, FArg p, int Vh, int nsub,
                                                     const int *active, double *partial, int pstride)
{
    typedef typename SpinorIO<SP>::real real;
    const int rid = active[blockIdx.y];
    const int s = blockIdx.x * kBlock + threadIdx.x;
    double nrm = 0.0;
    if (s < nsub * Vh) {
        const int sub = s / Vh, i = s - sub * Vh;
        double v[24];
        SpinorIO<SP_F64>::load(site_base(FRESH ? b : r, rid, sub), b.cs, i, v);
        if constexpr (FRESH) {
            double z[24];
#pragma unroll
            for (int k = 0; k < 24; k++) {
                nrm = fmaT(v[k], v[k], nrm);
                z[k] = 0.0;
            }
            SpinorIO<SP_F64>::store(site_base(r, rid, sub), r.cs, i, v);
            SpinorIO<SP_F64>::store(site_base(x, rid, sub), x.cs, i, z);
        }
        if constexpr (SP == SP_F64) {
            SpinorIO<SP_F64>::store(site_base(p, rid, sub), p.cs, i, v);
        } else {
            float z[24];
            real q[24], q2[24];
#pragma unroll
            for (int k = 0; k < 24; k++) z[k] = 0.f;
            SpinorIO<SP_F32>::store(site_base(xs, rid, sub), xs.cs, i, z);
            store_rt<SP>(site_base(rs, rid, sub), rs.cs, i, v, q);
            store_rt<SP>(site_base(p, rid, sub), p.cs, i, q, q2);
        }
    }
    if constexpr (FRESH) {
        nrm = sum16(nrm);
        if ((threadIdx.x & 15) == 0 && s < nsub * Vh) partial[(size_t)rid * pstride + (s >> 4)] = nrm;
    }
}

// Reliable update, before the FP64 sweeps: p -= r; SLOPPY: xhi += xs, xs = 0;
// the first work-group of a RHS keeps rr in rr_s.
template <int SP, int XP, bool SLOPPY>
__global__ void __launch_bounds__(kBlock) k_ru_begin(FArg p, FArg r, FArg xhi, FArg xs, const double *rr, double *rr_s,
                                                      int Vh, int nsub, const int *active)
{
    typedef typename SpinorIO<SP>::real real;
    const int rid = active[blockIdx.y];
    const int s = blockIdx.x * kBlock + threadIdx.x;
    if (s == 0) rr_s[rid] = rr[rid];
    if (s >= nsub * Vh) return;
    const int sub = s / Vh, i = s - sub * Vh;
    real pv[24], rv[24];
    SpinorIO<SP>::load(site_base(p, rid, sub), p.cs, i, pv);
    SpinorIO<SP>::load(site_base(r, rid, sub), r.cs, i, rv);
#pragma unroll
    for (int k = 0; k < 24; k++) pv[k] = fmaT((real)-1, rv[k], pv[k]);
    SpinorIO<SP>::store(site_base(p, rid, sub), p.cs, i, pv);
    if constexpr (SLOPPY) {
        double h[24], l[24];
        SpinorIO<SP_F64>::load(site_base(xhi, rid, sub), xhi.cs, i, h);
        SpinorIO<XP>::load(site_base(xs, rid, sub), xs.cs, i, l);
#pragma unroll
        for (int k = 0; k < 24; k++) {
            h[k] += l[k];
            l[k] = 0.0;
        }
        SpinorIO<SP_F64>::store(site_base(xhi, rid, sub), xhi.cs, i, h);
        SpinorIO<XP>::store(site_base(xs, rid, sub), xs.cs, i, l);
    }
}

// After the sweeps: SLOPPY: r = r64 in the sloppy format; partials of <r, p> =
// sum conj(r) p (r as stored).
template <int SP, bool SLOPPY>
__global__ void __launch_bounds__(kBlock) k_ru_mid(FArg r64, FArg r, FArg p, int Vh, int nsub, const int *active,
                                                    double *pre, double *pim, int pstride)
{
    typedef typename SpinorIO<SP>::real real;
    const int rid = active[blockIdx.y];
    const int s = blockIdx.x * kBlock + threadIdx.x;
    double vr = 0.0, vi = 0.0;
    if (s < nsub * Vh) {
        const int sub = s / Vh, i = s - sub * Vh;
        real x[24], y[24];
        if constexpr (SLOPPY) {
            double v[24];
            SpinorIO<SP_F64>::load(site_base(r64, rid, sub), r64.cs, i, v);
            store_rt<SP>(site_base(r, rid, sub), r.cs, i, v, x);
        } else {
            SpinorIO<SP>::load(site_base(r, rid, sub), r.cs, i, x);
        }
        SpinorIO<SP>::load(site_base(p, rid, sub), p.cs, i, y);
#pragma unroll
        for (int k = 0; k < 12; k++) {
            const double ar = x[2 * k], ai = x[2 * k + 1], br = y[2 * k], bi = y[2 * k + 1];
            vr = fmaT(ar, br, vr);
            vr = fmaT(ai, bi, vr);
            vi = fmaT(ar, bi, vi);
            vi = fmaT(-ai, br, vi);
        }
    }
    vr = sum16(vr);
    vi = sum16(vi);
    if ((threadIdx.x & 15) == 0 && s < nsub * Vh) {
        pre[(size_t)rid * pstride + (s >> 4)] = vr;
        pim[(size_t)rid * pstride + (s >> 4)] = vi;
    }
}

// Three sums a RHS (blockIdx.x = 0: |r|^2, 1: Re <r, p>, 2: Im).
__global__ void __launch_bounds__(kBlock) k_ru_sums(const double *prr, int nwr, const double *pre, const double *pim,
                                                     int nw, int pstride, double *rr, double *hout, double *dre,
                                                     double *dim, const int *active)
{
    __shared__ double sh[kBlock];
    const int rid = active[blockIdx.y], which = blockIdx.x;
    const double *pp = which == 0 ? prr : (which == 1 ? pre : pim);
    const double s = fin_block_sum(pp + (size_t)rid * pstride, which == 0 ? nwr : nw, sh);
    if (threadIdx.x != 0) return;
    if (which == 0) {
        rr[rid] = s;
        hout[rid] = s;
        __threadfence_system();
    } else {
        (which == 1 ? dre : dim)[rid] = s;
    }
}

// p -= c r with c = <r, p> / rr (complex), kept in p's format, then p = r +
// (rr / rr_s) p.
template <int SP>
__global__ void __launch_bounds__(kBlock) k_ru_end(FArg p, FArg r, const double *dre, const double *dim,
                                                    const double *rr, const double *rr_s, int Vh, int nsub,
                                                    const int *active)
{
    typedef typename SpinorIO<SP>::real real;
    const int rid = active[blockIdx.y];
    const int s = blockIdx.x * kBlock + threadIdx.x;
    if (s >= nsub * Vh) return;
    const int sub = s / Vh, i = s - sub * Vh;
    const double n = rr[rid], d = rr_s[rid];
    const real cr = (real)(n > 0.0 ? dre[rid] / n : 0.0), ci = (real)(n > 0.0 ? dim[rid] / n : 0.0);
    const real b = (real)(d > 0.0 ? n / d : 0.0);
    real pv[24], rv[24], q[24];
    SpinorIO<SP>::load(site_base(p, rid, sub), p.cs, i, pv);
    SpinorIO<SP>::load(site_base(r, rid, sub), r.cs, i, rv);
#pragma unroll
    for (int k = 0; k < 12; k++) {
        const real ar = rv[2 * k], ai = rv[2 * k + 1];
        pv[2 * k] = fmaT(-cr, ar, fmaT(ci, ai, pv[2 * k]));
        pv[2 * k + 1] = fmaT(-cr, ai, fmaT(-ci, ar, pv[2 * k + 1]));
    }
    if constexpr (has_norm(SP)) {
        uint32_t w[12];
        const float m = SpinorIO<SP>::encode(pv, w);
#pragma unroll
        for (int k = 0; k < 12; k++) SpinorIO<SP>::decode(w[k], m, &q[2 * k], &q[2 * k + 1]);
    } else {
#pragma unroll
        for (int k = 0; k < 24; k++) q[k] = pv[k];
    }
#pragma unroll
    for (int k = 0; k < 24; k++) q[k] = fmaT(b, q[k], rv[k]);
    SpinorIO<SP>::store(site_base(p, rid, sub), p.cs, i, q);
}

// One work-group per active RHS: fixed-order sum of its partials, then the
// CG scalar update selected by mode.
__global__ void __launch_bounds__(kBlock) k_finalize(const double *partial, int pstride, int nw,
                                                      const int *active, int mode, double *rr,
                                                      double *alpha, double *beta, double *out, double *hout)
{
    __shared__ double sh[kBlock];
    const int rid = active[blockIdx.x];
    const double s = fin_block_sum(partial + (size_t)rid * pstride, nw, sh);
    if (threadIdx.x == 0) {
        if (mode == FIN_STORE) {
            out[rid] = s;
        } else if (mode == FIN_ALPHA) {
            // s = p.Ap = |M p|^2; out: the iteration's slot of the alpha history
            fin_alpha_update(s, rid, rr, alpha, out);
        } else if (mode == FIN_BETA) {
            beta[rid] = s / rr[rid];
            rr[rid] = s;
        } else {
            rr[rid] = s;
            if (out) out[rid] = s;
        }
        if (hout) {
            hout[rid] = s;
            __threadfence_system();
        }
    }
}

inline dim3 grid_of(int Vh, int nsub, int nact) { return dim3((nsub * Vh + kBlock - 1) / kBlock, nact); }

}  // namespace

#define SP_SWITCH(sp, F)                                                                          \
    switch (sp) {                                                                                 \
    case SP_F64: F(SP_F64); break;                                                                \
    case SP_F32: F(SP_F32); break;                                                                \
    case SP_F16: F(SP_F16); break;                                                                \
    case SP_I16: F(SP_I16); break;                                                                \
    default: return hipErrorInvalidValue;                                                         \
    }

hipError_t blas_norm(const Field &a, int Vh, const int *active, int nact, double *partial,
                     int pstride, hipStream_t s)
{
    if (nact == 0) return hipSuccess;
#define F(SP) hipLaunchKernelGGL(k_norm<SP>, grid_of(Vh, a.nsub, nact), dim3(kBlock), 0, s, fa(a), Vh, a.nsub, active, partial, pstride)
    SP_SWITCH(a.sp, F)
#undef F
    return hipGetLastError();
}

hipError_t blas_p_update(const Field &p, const Field &r, const double *beta, int Vh,
                         const int *active, int nact, hipStream_t s)
{
    if (nact == 0) return hipSuccess;
    if (p.sp != r.sp) return hipErrorInvalidValue;
#define F(SP) hipLaunchKernelGGL(k_p_update<SP>, grid_of(Vh, p.nsub, nact), dim3(kBlock), 0, s, fa(p), fa(r), beta, Vh, p.nsub, active)
    SP_SWITCH(p.sp, F)
#undef F
    return hipGetLastError();
}

hipError_t blas_p_update_ring(const Field *p, int m, const Field &pdst, const Field &r, const BetaFold &bf,
                              double *beta, bool flush, const Field &x, const double *ahist, int ahs, int Vh,
                              const int *active, int nact, hipStream_t s)
{
    if (nact == 0) return hipSuccess;
    if (m < 1 || m > kMaxRing || pdst.nsub != 1) return hipErrorInvalidValue;
    Ring R{};
    for (int j = 0; j < m; j++) R.base[j] = p[j].base;
    R.rs = p[0].rs;
    const BetaArg bt{bf.partial, bf.pstride, bf.nw, bf.rr_in, bf.rr_out, beta, bf.hout};
    const dim3 grid = grid_of(Vh, 1, nact);
#define F(SP_, XP_)                                                                                       \
    if (flush)                                                                                            \
        hipLaunchKernelGGL((k_p_update_ring<SP_, XP_, true>), grid, dim3(kBlock), 0, s, R, m, fa(pdst), fa(r), \
                           bt, fa(x), ahist, ahs, Vh, active);                                            \
    else                                                                                                  \
        hipLaunchKernelGGL((k_p_update_ring<SP_, XP_, false>), grid, dim3(kBlock), 0, s, R, m, fa(pdst),     \
                           fa(r), bt, fa(x), ahist, ahs, Vh, active);
    if (pdst.sp == SP_F64 && (!flush || x.sp == SP_F64)) {
        F(SP_F64, SP_F64)
    } else if (pdst.sp != SP_F64 && (!flush || x.sp == SP_F32)) {
        switch (pdst.sp) {
        case SP_F32: F(SP_F32, SP_F32) break;
        case SP_F16: F(SP_F16, SP_F32) break;
        case SP_I16: F(SP_I16, SP_F32) break;
        default: return hipErrorInvalidValue;
        }
    } else {
        return hipErrorInvalidValue;
    }
#undef F
    return hipGetLastError();
}

hipError_t blas_cg_update(const Field &x, const Field &p, const Field &r, const Field &Ap,
                          const double *alpha, int Vh, const int *active, int nact,
                          double *partial, int pstride, hipStream_t s)
{
    if (nact == 0) return hipSuccess;
    dim3 gr = grid_of(Vh, p.nsub, nact);
    if (p.sp == SP_F64 && x.sp == SP_F64)
        hipLaunchKernelGGL((k_cg_update<SP_F64, SP_F64>), gr, dim3(kBlock), 0, s, fa(x), fa(p), fa(r), fa(Ap), alpha, Vh, p.nsub, active, partial, pstride);
    else if (p.sp == SP_F32 && x.sp == SP_F32)
        hipLaunchKernelGGL((k_cg_update<SP_F32, SP_F32>), gr, dim3(kBlock), 0, s, fa(x), fa(p), fa(r), fa(Ap), alpha, Vh, p.nsub, active, partial, pstride);
    else if (p.sp == SP_F16 && x.sp == SP_F32)
        hipLaunchKernelGGL((k_cg_update<SP_F16, SP_F32>), gr, dim3(kBlock), 0, s, fa(x), fa(p), fa(r), fa(Ap), alpha, Vh, p.nsub, active, partial, pstride);
    else if (p.sp == SP_I16 && x.sp == SP_F32)
        hipLaunchKernelGGL((k_cg_update<SP_I16, SP_F32>), gr, dim3(kBlock), 0, s, fa(x), fa(p), fa(r), fa(Ap), alpha, Vh, p.nsub, active, partial, pstride);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t blas_copy(const Field &dst, const Field &src, int Vh, const int *active, int nact,
                     hipStream_t s)
{
    if (nact == 0) return hipSuccess;
    if (dst.sp != src.sp) return hipErrorInvalidValue;
#define F(SP) hipLaunchKernelGGL(k_copy<SP>, grid_of(Vh, dst.nsub, nact), dim3(kBlock), 0, s, fa(dst), fa(src), Vh, dst.nsub, active)
    SP_SWITCH(dst.sp, F)
#undef F
    return hipGetLastError();
}

hipError_t blas_set_ids(int *dst, const int *ids, int n, hipStream_t s)
{
    for (int b = 0; b < n; b += 64) {
        IdList l;
        l.n = n - b < 64 ? n - b : 64;
        for (int q = 0; q < 64; q++) l.id[q] = q < l.n ? ids[b + q] : 0;
        hipLaunchKernelGGL(k_set_ids, dim3(1), dim3(64), 0, s, dst + b, l);
    }
    return hipGetLastError();
}

hipError_t blas_set_coefs(double *c1, double *c2, const int *ids, const double *kappa, int n, hipStream_t s)
{
    for (int b = 0; b < n; b += 32) {
        CoefList l;
        l.n = n - b < 32 ? n - b : 32;
        for (int q = 0; q < 32; q++) {
            l.id[q] = q < l.n ? ids[b + q] : 0;
            l.kappa[q] = q < l.n ? kappa[b + q] : 0.0;
        }
        hipLaunchKernelGGL(k_set_coefs, dim3(1), dim3(64), 0, s, c1, c2, l);
    }
    return hipGetLastError();
}

hipError_t blas_cg_init(bool fresh, const Field &b, const Field &x, const Field &r, const Field &rs, const Field &xs,
                        const Field &p, int Vh, const int *active, int nact, double *partial, int pstride,
                        hipStream_t s)
{
    if (nact == 0) return hipSuccess;
    const dim3 gr = grid_of(Vh, b.nsub, nact);
#define F(SP)                                                                                                     \
    if (fresh)                                                                                                    \
        hipLaunchKernelGGL((k_cg_init<SP, true>), gr, dim3(kBlock), 0, s, fa(b), fa(x), fa(r), fa(rs), fa(xs), fa(p), \
                           Vh, b.nsub, active, partial, pstride);                                                 \
    else                                                                                                          \
        hipLaunchKernelGGL((k_cg_init<SP, false>), gr, dim3(kBlock), 0, s, fa(b), fa(x), fa(r), fa(rs), fa(xs), fa(p), \
                           Vh, b.nsub, active, partial, pstride)
    SP_SWITCH(p.sp, F)
#undef F
    return hipGetLastError();
}

hipError_t blas_ru_begin(const Field &p, const Field &r, const Field &x, const Field *xs, const double *rr, double *rr_s,
                         int Vh, const int *active, int nact, hipStream_t s)
{
    if (nact == 0) return hipSuccess;
    if (p.sp != r.sp || (xs && xs->sp != SP_F32)) return hipErrorInvalidValue;
    const dim3 gr = grid_of(Vh, p.nsub, nact);
#define F(SP)                                                                                                        \
    if (xs)                                                                                                          \
        hipLaunchKernelGGL((k_ru_begin<SP, SP_F32, true>), gr, dim3(kBlock), 0, s, fa(p), fa(r), fa(x), fa(*xs), rr, rr_s, \
                           Vh, p.nsub, active);                                                                      \
    else                                                                                                             \
        hipLaunchKernelGGL((k_ru_begin<SP, SP_F32, false>), gr, dim3(kBlock), 0, s, fa(p), fa(r), fa(x), fa(x), rr, rr_s, \
                           Vh, p.nsub, active)
    SP_SWITCH(p.sp, F)
#undef F
    return hipGetLastError();
}

hipError_t blas_ru_mid(const Field &r64, const Field &r, bool sloppy, const Field &p, int Vh, const int *active,
                       int nact, double *pre, double *pim, int pstride, hipStream_t s)
{
    if (nact == 0) return hipSuccess;
    if (p.sp != r.sp) return hipErrorInvalidValue;
    const dim3 gr = grid_of(Vh, p.nsub, nact);
#define F(SP)                                                                                                     \
    if (sloppy)                                                                                                   \
        hipLaunchKernelGGL((k_ru_mid<SP, true>), gr, dim3(kBlock), 0, s, fa(r64), fa(r), fa(p), Vh, p.nsub, active, pre, \
                           pim, pstride);                                                                         \
    else                                                                                                          \
        hipLaunchKernelGGL((k_ru_mid<SP, false>), gr, dim3(kBlock), 0, s, fa(r64), fa(r), fa(p), Vh, p.nsub, active, pre, \
                           pim, pstride)
    SP_SWITCH(p.sp, F)
#undef F
    return hipGetLastError();
}

hipError_t blas_ru_sums(const double *prr, int nwr, const double *pre, const double *pim, int nw, int pstride,
                        double *rr, double *hout, double *dre, double *dim, const int *active, int nact,
                        hipStream_t s)
{
    if (nact == 0) return hipSuccess;
    hipLaunchKernelGGL(k_ru_sums, dim3(3, nact), dim3(kBlock), 0, s, prr, nwr, pre, pim, nw, pstride, rr, hout, dre, dim,
                       active);
    return hipGetLastError();
}

hipError_t blas_ru_end(const Field &p, const Field &r, const double *dre, const double *dim, const double *rr,
                       const double *rr_s, int Vh, const int *active, int nact, hipStream_t s)
{
    if (nact == 0) return hipSuccess;
    if (p.sp != r.sp) return hipErrorInvalidValue;
#define F(SP) hipLaunchKernelGGL(k_ru_end<SP>, grid_of(Vh, p.nsub, nact), dim3(kBlock), 0, s, fa(p), fa(r), dre, dim, rr, rr_s, Vh, p.nsub, active)
    SP_SWITCH(p.sp, F)
#undef F
    return hipGetLastError();
}

hipError_t blas_finalize(const double *partial, int pstride, int nw, const int *active, int nact,
                         int mode, double *rr, double *alpha, double *beta, double *out, double *hout,
                         hipStream_t s)
{
    if (nact == 0) return hipSuccess;
    hipLaunchKernelGGL(k_finalize, dim3(nact), dim3(kBlock), 0, s, partial, pstride, nw, active, mode, rr, alpha, beta, out, hout);
    return hipGetLastError();
}

}  // namespace wd
