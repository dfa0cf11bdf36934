// cg_small.hip -- FP64 conjugate gradient on lattices that fit one work-group.
//
// On 4^4 an iteration of the general path is 6 (even-odd) or 8 (full lattice)
// dependent launches of 2-6 us, each a microsecond or less of work, and the
// host reads the residual every few iterations.  Here one work-group per
// right-hand side runs whole steps of the solver: two lanes per site
// (half_spinor.h) keep p, r and x in registers, the vector whose neighbours
// the next sweep reads goes through LDS, and the scalars are summed from LDS
// by every wave for itself.  The values, their order and roundings are those
// of the general path's kernels, bit for bit.
//
// Bound by instruction issue on one CU: a full-lattice 4^4 iteration is about
// 2100 instructions in each of two waves a SIMD (980 of them FP64), 7 us at four
// cycles each, and takes 9.2 us.  The links (295 KB a sweep, 18-real) would cost
// as much again if each half loaded all of them, hence load_link_halves.  Full
// 4^4 solve to 1e-12, 168 iterations: 6.69 ms with the general path, 39.8 us an
// iteration; 1.5 ms in this kernel.
//
// A launch takes as many right-hand sides as there are CUs (the LDS holds one
// work-group a CU; the id lists, 2 KB, are kernel arguments).  Even-odd 4^4
// solves to 1e-12 of 256 and 1000 right-hand sides: 4.4 and 13.0 ms with the
// general path, 5.1 and 20.4 with launches of 32 one after the other, 0.90 and
// 3.7 with 256; 2^3 x 4 with 1000: 9.0, 24.0 and 3.4.
#include <cmath>

#include "half_spinor.h"
#include "wd_internal.h"

namespace wd {

namespace {

// Vectors in LDS: chunk stride kSmallSites whatever the lattice, so that a
// row's words are at constant offsets.
typedef __attribute__((address_space(3))) dbl2_t lds2_t;
constexpr int kLdsVec = 12 * kSmallSites;

struct LdsRows {
    const lds2_t *f;
    __device__ __forceinline__ void operator()(int r, int j, double v[6]) const { load_row64(f, kSmallSites, r, j, v); }
};

// The site index of a sweep, opaque to the compiler: neighbour indexes and link
// addresses are formed where they are used, not hoisted out of the iteration
// loop, where they would not fit the registers.
__device__ __forceinline__ int here(int i)
{
    asm volatile("" : "+v"(i));
    return i;
}

// The hopping term of the lane's site i of parity P (half_spinor.h).
template <int LK, bool DAG>
__device__ __forceinline__ void sweep_half(const SmallArgs &a, int P, int i0, int half, const LdsRows &nb, double acc1[6],
                                           double acc2[6])
{
    const int i = here(i0);
    int c[4];
    site_coords(a.g, i, P, c);
    hop_half_all<LK, DAG>(a.links, a.g, P, i, c, half, nb, acc1, acc2);
}

// Partial sums of 16 sites, then every wave adds the n <= 64 of them in the
// order of the finalize kernels (a halving tree over zero-padded lanes).
__device__ __forceinline__ void put_leaf(double nrm, int site, double *leaf)
{
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) nrm += __shfl_xor(nrm, off, 64);
    if (((int)threadIdx.x & 63) >= 32 && (site & 15) == 0) leaf[site >> 4] = nrm;
}
__device__ __forceinline__ double sum_leaves(const double *leaf, int n)
{
    const int lane = (int)threadIdx.x & 63;
    double v = lane < n ? leaf[lane] : 0.0;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

static_assert(sizeof(SmallArgs) <= 4096, "kernel arguments");

// One work-group per right-hand side, 64 threads per 32 sites (Vh sites, or 2
// Vh on the full lattice).
template <int LK, bool EO>
__global__ void __launch_bounds__(2 * kSmallSites) k_cg_small(SmallArgs a)
{
    extern __shared__ __attribute__((aligned(16))) char small_lds[];
    __shared__ double leaves[2][kSmallSites / 16];
    const int slot = blockIdx.x, rid = a.rid[slot];
    const Geom &g = a.g;
    const int n = EO ? g.Vh : 2 * g.Vh, nleaf = n >> 4;
    const int lane = (int)threadIdx.x & 63, half = lane >> 5;
    const int s = (int)(threadIdx.x >> 6) * 32 + (lane & 31);  // the lane's site
    const int sub = (!EO && s >= g.Vh) ? 1 : 0, i = s - sub * g.Vh;
    // (n is a multiple of 16: a wave may be half idle, but not a group of 16)
    const bool live = s < n;
    lds2_t *V0 = (lds2_t *)small_lds;  // p, and with EO t
    lds2_t *V1 = V0 + kLdsVec;         // EO: the odd vector; full: t
    const int r2 = 2 + half;
    const double cf = a.coef[rid];
    double rr = a.rr[rid], alpha = 0.0, beta = 0.0;
    double p1[6], p2[6], r1[6], rv2[6], x1[6], x2[6];
    const dbl2_t *gp = reinterpret_cast<const dbl2_t *>(a.p.base + rid * a.p.rs + sub * a.p.ss);
    const dbl2_t *gr = reinterpret_cast<const dbl2_t *>(a.r.base + rid * a.r.rs + sub * a.r.ss);
    const dbl2_t *gx = reinterpret_cast<const dbl2_t *>(a.x.base + rid * a.x.rs + sub * a.x.ss);
    if (live) {
        load_row64(gp, g.cs, half, i, p1);
        load_row64(gp, g.cs, r2, i, p2);
        load_row64(gr, g.cs, half, i, r1);
        load_row64(gr, g.cs, r2, i, rv2);
        load_row64(gx, g.cs, half, i, x1);
        load_row64(gx, g.cs, r2, i, x2);
        store_row64(V0, kSmallSites, half, s, p1);
        store_row64(V0, kSmallSites, r2, s, p2);
    }
    __syncthreads();
    const double stop = a.tol2 * a.bb[rid];
    int it = a.it[slot];
    for (int step = 0; step < a.max_steps; step++) {
        const int k = a.maxiter - it < a.k ? a.maxiter - it : a.k;
        for (int q = 0; q < k; q++) {
            double acc1[6], acc2[6], t1[6], t2[6], nrm = 0.0;
            if constexpr (EO) {
                if (live) {  // to = D_oe p
                    sweep_half<LK, false>(a, 1, i, half, LdsRows{V0}, acc1, acc2);
                    store_row64(V1, kSmallSites, half, s, acc1);
                    store_row64(V1, kSmallSites, r2, s, acc2);
                }
                __syncthreads();
                if (live) {  // t = p + cf D_eo to
                    sweep_half<LK, false>(a, 0, i, half, LdsRows{V1}, acc1, acc2);
#pragma unroll
                    for (int e = 0; e < 6; e++) {
                        t1[e] = fmaT(cf, acc1[e], p1[e]);
                        t2[e] = fmaT(cf, acc2[e], p2[e]);
                    }
                    store_row64(V0, kSmallSites, half, s, t1);
                    store_row64(V0, kSmallSites, r2, s, t2);
                    nrm = half_norm(t1, t2);
                    put_leaf(nrm, s, leaves[0]);
                }
                __syncthreads();
                if (live) {  // to = D_oe^dag t
                    sweep_half<LK, true>(a, 1, i, half, LdsRows{V0}, acc1, acc2);
                    store_row64(V1, kSmallSites, half, s, acc1);
                    store_row64(V1, kSmallSites, r2, s, acc2);
                }
                __syncthreads();
                if (live) sweep_half<LK, true>(a, 0, i, half, LdsRows{V1}, acc1, acc2);
            } else {
                const int oth = (1 - sub) * g.Vh;
                if (live) {  // t = M p = p + cf H p
                    sweep_half<LK, false>(a, sub, i, half, LdsRows{V0 + oth}, acc1, acc2);
#pragma unroll
                    for (int e = 0; e < 6; e++) {
                        t1[e] = fmaT(cf, acc1[e], p1[e]);
                        t2[e] = fmaT(cf, acc2[e], p2[e]);
                    }
                    store_row64(V1, kSmallSites, half, s, t1);
                    store_row64(V1, kSmallSites, r2, s, t2);
                    nrm = half_norm(t1, t2);
                    put_leaf(nrm, s, leaves[0]);
                }
                __syncthreads();
                if (live) sweep_half<LK, true>(a, sub, i, half, LdsRows{V1 + oth}, acc1, acc2);
            }
            // alpha = rr / |t|^2 (as fin_alpha_update)
            const double pap = sum_leaves(leaves[0], nleaf);
            if (pap > 0.0 && pap < INFINITY) {
                alpha = rr / pap;
            } else {
                alpha = 0.0;
                rr = NAN;
            }
            if (live) {  // x += alpha p; r -= alpha (t + cf D^dag to)
#pragma unroll
                for (int e = 0; e < 6; e++) {
                    x1[e] = fmaT(alpha, p1[e], x1[e]);
                    x2[e] = fmaT(alpha, p2[e], x2[e]);
                    r1[e] = fmaT(-alpha, fmaT(cf, acc1[e], t1[e]), r1[e]);
                    rv2[e] = fmaT(-alpha, fmaT(cf, acc2[e], t2[e]), rv2[e]);
                }
                nrm = half_norm(r1, rv2);
                put_leaf(nrm, s, leaves[1]);
            }
            __syncthreads();
            const double rn = sum_leaves(leaves[1], nleaf);
            beta = rn / rr;
            rr = rn;
            if (live) {  // p = r + beta p
#pragma unroll
                for (int e = 0; e < 6; e++) {
                    p1[e] = fmaT(beta, p1[e], r1[e]);
                    p2[e] = fmaT(beta, p2[e], rv2[e]);
                }
                store_row64(V0, kSmallSites, half, s, p1);
                store_row64(V0, kSmallSites, r2, s, p2);
            }
            __syncthreads();
        }
        it += k;
        // (the same value in every lane: the host's test after a step)
        if (!(rr > stop) || !(rr < INFINITY) || it >= a.maxiter) break;
    }
    if (live) {
        store_row64(const_cast<dbl2_t *>(gp), g.cs, half, i, p1);
        store_row64(const_cast<dbl2_t *>(gp), g.cs, r2, i, p2);
        store_row64(const_cast<dbl2_t *>(gr), g.cs, half, i, r1);
        store_row64(const_cast<dbl2_t *>(gr), g.cs, r2, i, rv2);
        store_row64(const_cast<dbl2_t *>(gx), g.cs, half, i, x1);
        store_row64(const_cast<dbl2_t *>(gx), g.cs, r2, i, x2);
    }
    if (threadIdx.x == 0) {
        a.rr[rid] = rr;
        a.alpha[rid] = alpha;
        a.beta[rid] = beta;
        a.it_out[rid] = it;
        a.hout[rid] = rr;
        __threadfence_system();
    }
}

}  // namespace

bool cg_small_ok(const Geom &g, int nsub) { return g.Vh % 16 == 0 && nsub * g.Vh <= kSmallSites; }

hipError_t cg_small_launch(const SmallArgs &a, int nrhs, int lk, bool eo, hipStream_t s)
{
    const int n = eo ? a.g.Vh : 2 * a.g.Vh;
    const dim3 grid(nrhs), block((n + 31) / 32 * 64);
    constexpr unsigned lds = 2 * kLdsVec * sizeof(dbl2_t);
#define SMALL(LK_, EO_)                                                                                             \
    if (lk == LK_ && eo == EO_) {                                                                                   \
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_cg_small<LK_, EO_>),             \
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);             \
        if (e != hipSuccess) return e;                                                                              \
        hipLaunchKernelGGL((k_cg_small<LK_, EO_>), grid, block, lds, s, a);                                         \
        return hipGetLastError();                                                                                   \
    }
    SMALL(LK_F64_18, true)
    SMALL(LK_F64_18, false)
    SMALL(LK_F64_12, true)
    SMALL(LK_F64_12, false)
#undef SMALL
    return hipErrorInvalidValue;
}

}  // namespace wd
