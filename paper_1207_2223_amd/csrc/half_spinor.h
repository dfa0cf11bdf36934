// half_spinor.h -- the hopping term with two lanes per site: lane 0-31 of a
// wave carry spin row 0 of the half spinors of 32 sites, lanes 32-63 row 1 of
// the same sites, with half the registers and half the dependent instructions
// of one lane per site.
//
// (1 + S g_mu) psi has the rows h_0, h_1 (wd_device.h); lane half a needs rows
// a and b of psi, b = 3 - a for x and y and b = 2 + a for z and t, and the
// rebuilt spinor adds to rows a and b.  Both are of one form with a sign s:
//   x: h = p_a + S i p_b,    row b -= S i h        (z with S -> s S, s = 1, -1)
//   y: h = p_a + s S p_b,    row b += s S h        (s = -1, 1)
//   t: h = p_a + S p_b,      row b += S h
// so each lane runs the same instructions.  The sums over the directions keep
// the order of one lane per site: between y and z the halves exchange the
// second accumulator (rows 3 | 2 become 2 | 3).  Products with a sign are
// exact, so every value has the roundings of dslash_kernel.
#pragma once

#include "wd_device.h"

namespace wd {

// Row r (0..3) of the FP64 spinor of site j in a structure of arrays (chunk
// stride cs): three consecutive chunks.
template <class P>
__device__ __forceinline__ void load_row64(P f, int cs, int r, int j, double v[6])
{
    f += 3 * r * cs + j;
#pragma unroll
    for (int k = 0; k < 3; k++) {
        const dbl2_t w = f[k * cs];
        v[2 * k] = w.x;
        v[2 * k + 1] = w.y;
    }
}
template <class P>
__device__ __forceinline__ void store_row64(P f, int cs, int r, int j, const double v[6])
{
    f += 3 * r * cs + j;
#pragma unroll
    for (int k = 0; k < 3; k++) f[k * cs] = dbl2_t{v[2 * k], v[2 * k + 1]};
}

// A 16-byte word of each half to both: lanes 0-31 hold word a of their sites,
// lanes 32-63 word b of the same sites.
__device__ __forceinline__ void both_halves(dbl2_t w, dbl2_t &a, dbl2_t &b)
{
    const u32x4_t x = __builtin_bit_cast(u32x4_t, w);
    u32x4_t lo, hi;
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const auto s = __builtin_amdgcn_permlane32_swap(x[k], x[k], false, false);
        lo[k] = s[0];
        hi[k] = s[1];
    }
    a = __builtin_bit_cast(dbl2_t, lo);
    b = __builtin_bit_cast(dbl2_t, hi);
}

// The link of both halves of a site, each half loading half of it: the loads
// of one CU are its narrowest part here (64 bytes a clock).
template <int LK>
__device__ __forceinline__ void load_link_halves(const char *U, int cs, int blk, int i, int half, double u[18])
{
    // (scalar bases and one 32-bit lane offset: the links of these lattices
    // are far below 4 GiB; a wave may hold both parities, so blk is a lane's)
    constexpr int nch = LK == LK_F64_18 ? 9 : 6, h = nch / 2;
    const uint32_t own = pin_v((uint32_t)((blk * nch + half * h) * cs + i) * 16u);
    dbl2_t w[h];
#pragma unroll
    for (int k = 0; k < h; k++) w[k] = ld_off<dbl2_t, true>(U + (size_t)k * cs * 16, own);
    dbl2_t e{};
    if constexpr (LK == LK_F64_18)
        e = ld_off<dbl2_t, true>(U + (size_t)8 * cs * 16, pin_v((uint32_t)(blk * nch * cs + i) * 16u));
#pragma unroll
    for (int k = 0; k < h; k++) {
        dbl2_t a, b;
        both_halves(w[k], a, b);
        u[2 * k] = a.x;
        u[2 * k + 1] = a.y;
        u[2 * (h + k)] = b.x;
        u[2 * (h + k) + 1] = b.y;
    }
    if constexpr (LK == LK_F64_18) {
        u[16] = e.x;
        u[17] = e.y;
    } else {
        reconstruct_row3(u);
    }
}

// One term of direction MU: h = the lane's projected row from rows a (pa) and
// b (pb); w = U h or U^dag h; acc1 += w, acc2 += its rebuilt partner.  sg: the
// sign s S above.
template <int MU, bool ADJ, typename T>
__device__ __forceinline__ void hop_half(const T u[18], const T pa[6], const T pb[6], T sg, T acc1[6], T acc2[6])
{
    T h[6];
#pragma unroll
    for (int c = 0; c < 3; c++) {
        if (MU == 0 || MU == 2) {
            h[2 * c] = fmaT(-sg, pb[2 * c + 1], pa[2 * c]);
            h[2 * c + 1] = fmaT(sg, pb[2 * c], pa[2 * c + 1]);
        } else {
            h[2 * c] = fmaT(sg, pb[2 * c], pa[2 * c]);
            h[2 * c + 1] = fmaT(sg, pb[2 * c + 1], pa[2 * c + 1]);
        }
    }
#pragma unroll
    for (int a = 0; a < 3; a++) {
        T re = 0, im = 0;
#pragma unroll
        for (int b = 0; b < 3; b++) {
            const int idx = ADJ ? 2 * (3 * b + a) : 2 * (3 * a + b);
            const T ur = u[idx], ui = ADJ ? -u[idx + 1] : u[idx + 1];
            re = fmaT(ur, h[2 * b], re);
            re = fmaT(-ui, h[2 * b + 1], re);
            im = fmaT(ur, h[2 * b + 1], im);
            im = fmaT(ui, h[2 * b], im);
        }
        acc1[2 * a] += re;
        acc1[2 * a + 1] += im;
        if (MU == 0 || MU == 2) {
            acc2[2 * a] = fmaT(sg, im, acc2[2 * a]);
            acc2[2 * a + 1] = fmaT(-sg, re, acc2[2 * a + 1]);
        } else {
            acc2[2 * a] = fmaT(sg, re, acc2[2 * a]);
            acc2[2 * a + 1] = fmaT(sg, im, acc2[2 * a + 1]);
        }
    }
}

// The hopping term of output site i (parity P, coordinates c) for lane half
// `half`: acc1 = row half, acc2 = row 2 + half.  nb(r, j, v): row r of input
// site j.
template <int MU, int LK, bool DAG, class NB>
__device__ __forceinline__ void hop_half_dir(const char *links, const Geom &g, int P, int i, const int c[4], int half,
                                             const NB &nb, double acc1[6], double acc2[6])
{
    constexpr int SF = DAG ? +1 : -1;  // forward: (1 - g) for H, (1 + g) for H^dag
    const double s = MU == 1 ? (half ? 1.0 : -1.0) : (MU == 2 && half ? -1.0 : 1.0);
    const int b = MU < 2 ? 3 - half : 2 + half;
    double u[18], pa[6], pb[6];
    {
        const int j = neighbour<MU, +1>(g, i, c);
        load_link_halves<LK>(links, g.cs, P * 4 + MU, i, half, u);
        nb(half, j, pa);
        nb(b, j, pb);
        hop_half<MU, false>(u, pa, pb, s * SF, acc1, acc2);
    }
    {
        const int j = neighbour<MU, -1>(g, i, c);
        load_link_halves<LK>(links, g.cs, (1 - P) * 4 + MU, j, half, u);
        nb(half, j, pa);
        nb(b, j, pb);
        hop_half<MU, true>(u, pa, pb, -s * SF, acc1, acc2);
    }
}
template <int LK, bool DAG, class NB>
__device__ __forceinline__ void hop_half_all(const char *links, const Geom &g, int P, int i, const int c[4], int half,
                                             const NB &nb, double acc1[6], double acc2[6])
{
#pragma unroll
    for (int k = 0; k < 6; k++) acc1[k] = acc2[k] = 0.0;
    hop_half_dir<0, LK, DAG>(links, g, P, i, c, half, nb, acc1, acc2);
    hop_half_dir<1, LK, DAG>(links, g, P, i, c, half, nb, acc1, acc2);
#pragma unroll
    for (int k = 0; k < 6; k++) acc2[k] = __shfl_xor(acc2[k], 32, 64);
    hop_half_dir<2, LK, DAG>(links, g, P, i, c, half, nb, acc1, acc2);
    hop_half_dir<3, LK, DAG>(links, g, P, i, c, half, nb, acc1, acc2);
}

// Sum of the squares of a site's 24 reals, added in the order of one lane per
// site (rows 0, 1, 2, 3): v1 = row half, v2 = row 2 + half.  Valid in the
// lanes of half 1.
template <typename T>
__device__ __forceinline__ double half_norm(const T v1[6], const T v2[6])
{
    double s = 0.0;
#pragma unroll
    for (int ph = 0; ph < 4; ph++) {
        if (ph) s = __shfl_xor(s, 32, 64);
#pragma unroll
        for (int k = 0; k < 6; k++) {
            const double x = (double)(ph < 2 ? v1[k] : v2[k]);
            s = fmaT(x, x, s);
        }
    }
    return s;
}

}  // namespace wd
