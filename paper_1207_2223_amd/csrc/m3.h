// m3.h -- 3x3 complex matrices of the canonical link layout ([V][4][3][3]
// complex128) for the kernels that work on it: the molecular dynamics and the
// gauge measurements.
#pragma once

#include "wd_device.h"

namespace wd {

struct M3 {
    double2 e[9];  // row-major
};

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
// s + a b and s + a conj(b)
__device__ __forceinline__ double2 cfma(double2 a, double2 b, double2 s)
{
    return make_double2(fmaT(-a.y, b.y, fmaT(a.x, b.x, s.x)), fmaT(a.y, b.x, fmaT(a.x, b.y, s.y)));
}
__device__ __forceinline__ double2 cfmac(double2 a, double2 b, double2 s)
{
    return make_double2(fmaT(a.y, b.y, fmaT(a.x, b.x, s.x)), fmaT(a.y, b.x, fmaT(-a.x, b.y, s.y)));
}

__device__ __forceinline__ M3 load_m3(const double *p)
{
    M3 m;
    const double2 *q = reinterpret_cast<const double2 *>(p);
#pragma unroll
    for (int k = 0; k < 9; k++) m.e[k] = q[k];
    return m;
}
__device__ __forceinline__ void store_m3(double *p, const M3 &m)
{
    double2 *q = reinterpret_cast<double2 *>(p);
#pragma unroll
    for (int k = 0; k < 9; k++) q[k] = m.e[k];
}
__device__ __forceinline__ M3 mul(const M3 &a, const M3 &b)
{
    M3 c;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) {
            double2 s = make_double2(0, 0);
#pragma unroll
            for (int k = 0; k < 3; k++) s = cfma(a.e[3 * i + k], b.e[3 * k + j], s);
            c.e[3 * i + j] = s;
        }
    return c;
}
// a b^dag
__device__ __forceinline__ M3 mul_dag(const M3 &a, const M3 &b)
{
    M3 c;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) {
            double2 s = make_double2(0, 0);
#pragma unroll
            for (int k = 0; k < 3; k++) s = cfmac(a.e[3 * i + k], b.e[3 * j + k], s);
            c.e[3 * i + j] = s;
        }
    return c;
}

// Links read by a wave together.  A lane that reads its own link takes nine
// 16-byte words 144 bytes from the next lane's, each load touching 64 cache
// lines, and holds 36 registers a matrix, so that products of a few matrices
// leave one or two waves a SIMD.  Here three lanes share a link (21 links a
// wave, kRowLinks): the wave reads its links in memory order into 3 KB of LDS
// of its own, a lane keeps one row of the running product and takes the other
// factor from LDS.
constexpr int kRowLinks = 21;
constexpr int kRowWords = (kRowLinks + 1) * 9;  // (lane 63 has no link: it reads the unused last one)

struct Row3 {
    double2 e[3];
};

// The words of a wave's links on their way to LDS: several are fetched before
// the first is used, because a chain of fetch, product, fetch would wait for
// memory at every factor.  link: the same in the three lanes of a link, an
// element of U in any case; every lane of the wave takes part.
struct LinkWords {
    dbl2_t w[3];
};
__device__ __forceinline__ LinkWords fetch_links(const double *U, int link)
{
    const int lane = (int)threadIdx.x & 63;
    LinkWords f;
#pragma unroll
    for (int q = 0; q < 3; q++) {
        const int e = q * 64 + lane < kRowLinks * 9 ? q * 64 + lane : kRowLinks * 9 - 1, l = e / 9;
        const int src = __shfl(link, 3 * l, 64);
        f.w[q] = *reinterpret_cast<const dbl2u_t *>(U + (size_t)src * 18 + 2 * (e - 9 * l));
    }
    return f;
}
// (what lds held before has been read by then)
__device__ __forceinline__ void stage_links(const LinkWords &f, dbl2_t *lds)
{
    const int lane = (int)threadIdx.x & 63;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int q = 0; q < 3; q++)
        if (q * 64 + lane < kRowLinks * 9) lds[q * 64 + lane] = f.w[q];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
// The lane's row of its staged link.
__device__ __forceinline__ Row3 staged_row(const dbl2_t *lds)
{
    const int lane = (int)threadIdx.x & 63;
    Row3 r;
#pragma unroll
    for (int k = 0; k < 3; k++) {
        const dbl2_t w = lds[lane * 3 + k];
        r.e[k] = make_double2(w.x, w.y);
    }
    return r;
}
// Row a times the lane's staged link, or times its adjoint.
__device__ __forceinline__ Row3 row_mul(const Row3 &a, const dbl2_t *lds)
{
    const dbl2_t *m = lds + ((int)threadIdx.x & 63) / 3 * 9;
    Row3 r;
#pragma unroll
    for (int j = 0; j < 3; j++) r.e[j] = make_double2(0, 0);
#pragma unroll
    for (int k = 0; k < 3; k++)
#pragma unroll
        for (int j = 0; j < 3; j++) {
            const dbl2_t w = m[3 * k + j];
            r.e[j] = cfma(a.e[k], make_double2(w.x, w.y), r.e[j]);
        }
    return r;
}
__device__ __forceinline__ Row3 row_mul_dag(const Row3 &a, const dbl2_t *lds)
{
    const dbl2_t *m = lds + ((int)threadIdx.x & 63) / 3 * 9;
    Row3 r;
#pragma unroll
    for (int j = 0; j < 3; j++) {
        r.e[j] = make_double2(0, 0);
#pragma unroll
        for (int k = 0; k < 3; k++) {
            const dbl2_t w = m[3 * j + k];
            r.e[j] = cfmac(a.e[k], make_double2(w.x, w.y), r.e[j]);
        }
    }
    return r;
}

}  // namespace wd
