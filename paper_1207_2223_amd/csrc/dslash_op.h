// dslash_op.h -- one hopping sweep on canonical fields in one launch: the
// operator-level calls (wd_dslash, wd_mdagm) and the molecular dynamics read
// and write complex128 fields in the caller's layout, so the first sweep of a
// call can read them there and the last one write them there, instead of
// packing to the structure-of-arrays layout before and unpacking after.
//
// The sum, its order and the roundings of a format are those of dslash_kernel
// and of the pack and unpack kernels (the neighbour is encoded to the storage
// format as it is read, the result as it is written), so the results are the
// bits of pack, sweep, unpack.
#pragma once

#include "dslash_impl.h"

namespace wd {

// Source of the terms' spinors: the canonical complex128 field, 24 consecutive
// doubles a site.  full: lex order of the whole lattice (site 2 * cb + the low
// bit of x), else the cb order of one parity.  A neighbour is encoded to the
// storage format as it is used.
struct CanonRaw { dbl2u_t w[12]; };

template <int SP, int NR>
struct CanonNb {
    const CanonRaw (&s)[NR];

    template <typename real>
    __device__ __forceinline__ void values(int r, real v[24]) const
    {
#pragma unroll
        for (int k = 0; k < 12; k++) {
            v[2 * k] = (real)s[r].w[k].x;
            v[2 * k + 1] = (real)s[r].w[k].y;
        }
    }
    template <int MU, int DIR>
    __device__ __forceinline__ float half(const DslashArgs &, int, int r, int, _Float16 v[24]) const
    {
        double d[24];
        uint32_t w[12];
        values(r, d);
        const float m = SpinorIO<SP_F16>::encode(d, w);
#pragma unroll
        for (int k = 0; k < 12; k++) {
            v[2 * k] = __builtin_bit_cast(_Float16, (unsigned short)(w[k] & 0xffffu));
            v[2 * k + 1] = __builtin_bit_cast(_Float16, (unsigned short)(w[k] >> 16));
        }
        return m;
    }
    template <int MU, int DIR>
    __device__ __forceinline__ float h2(const DslashArgs &, int, int r, int, h2_t v[12]) const
    {
        double d[24];
        uint32_t w[12];
        values(r, d);
        const float m = SpinorIO<SP_F16>::encode(d, w);
#pragma unroll
        for (int k = 0; k < 12; k++) v[k] = __builtin_bit_cast(h2_t, w[k]);
        return m;
    }
    template <int MU, int DIR>
    __device__ __forceinline__ float i16(const DslashArgs &, int, int r, int, int v[24]) const
    {
        double d[24];
        uint32_t w[12];
        values(r, d);
        const float m = SpinorIO<SP_I16>::encode(d, w);
#pragma unroll
        for (int k = 0; k < 12; k++) {
            v[2 * k] = (int)(short)(w[k] & 0xffffu);
            v[2 * k + 1] = (int)(short)(w[k] >> 16);
        }
        return SpinorIO<SP_I16>::step(m);
    }
    template <int MU, int DIR, int SP_, typename real>
    __device__ __forceinline__ real gen(const DslashArgs &, int, int r, int, real v[24]) const
    {
        values(r, v);
        return (real)1;
    }
};

template <int SP>
struct CanonSrc {
    const double *base;
    bool full;
    int xbit;  // low bit of the output site's x

    typedef CanonRaw Raw;
    template <int NR> using Nb = CanonNb<SP, NR>;
    template <int MU>
    __device__ __forceinline__ void fetch(const DslashArgs &, int, int j, Raw &R) const
    {
        const long long site = full ? 2LL * j + (MU == 0 ? xbit ^ 1 : xbit) : (long long)j;
        const dbl2u_t *p = reinterpret_cast<const dbl2u_t *>(base + site * 24);
#pragma unroll
        for (int k = 0; k < 12; k++) R.w[k] = p[k];
    }
};

// The reals of an output spinor as the storage format keeps them.
template <int SP, typename real>
__device__ __forceinline__ void stored_values(const real v[24], double d[24])
{
    if constexpr (has_norm(SP)) {
        uint32_t w[12];
        const float n = SpinorIO<SP>::encode(v, w);
#pragma unroll
        for (int k = 0; k < 12; k++) {
            float lo, hi;
            SpinorIO<SP>::decode(w[k], n, &lo, &hi);
            d[2 * k] = (double)lo;
            d[2 * k + 1] = (double)hi;
        }
    } else {
#pragma unroll
        for (int k = 0; k < 24; k++) d[k] = (double)v[k];
    }
}

// One lane per output site; grid.x: the tiles of np parities (both parities
// of a tile one after the other on the same XCD: their input is each other's
// neighbourhood), grid.y: right-hand sides.  Work-groups of one wavefront:
// small lattices spread over more CUs, and at 24^3 x 24 and above 64 threads
// are still 2-5 % faster than 128.  CIN: neighbours (and the xpay operand)
// from the canonical field, else from the structure of arrays; the host's
// rule is op_reads_canonical.  Two terms are in flight from the canonical
// field (48 registers each for the spinor).  A call is bound by its launches
// up to about 12^3 x 24 and by the links' bytes above.  Against pack, sweep and
// unpack with uploads of ids and coefficients, then with terms fetched ahead:
// FP64 D_eo on 4^4 36.8 -> 10.2 -> 10 us a call, Mhat^dag Mhat on 16^3 x 32 119
// -> 66 -> 64, FP64 18-real D_oe^dag on 32^3 x 64 572 -> 412 -> 374 (1.6 GB, 4.3
// TB/s).
template <int SP, int LK, bool DAG, bool CIN>
__global__ void __launch_bounds__(256) dslash_op_kernel(OpArgs o)
{
    typedef typename SpinorIO<SP>::real real;
    const int L = xcd_remap((int)blockIdx.x, (int)gridDim.x);
    const int tile = o.np == 2 ? L >> 1 : L;
    const int P = o.np == 2 ? L & 1 : o.P0;
    const int i0 = tile * (int)blockDim.x + (int)threadIdx.x;
    const bool live = i0 < o.g.Vh;
    const int i = live ? i0 : o.g.Vh - 1;  // (lanes past the end compute the last site and store nothing)
    const long long rid = blockIdx.y;
    DslashArgs a;
    a.g = o.g;
    a.P = P;
    a.links = o.links;
    a.in_rs = 0;
    int c[4];
    site_coords(o.g, i, P, c);
    const long long site = o.full ? 2LL * i + (c[0] & 1) : (long long)i;
    const int one[1] = {0};
    real acc[1][24];
    if constexpr (CIN) {
        a.in = nullptr;
        const CanonSrc<SP> src{reinterpret_cast<const double *>(o.in) + rid * o.in_rs, o.full != 0, c[0] & 1};
        hop_ahead<2, SP, LK, 1, DAG>(a, src, one, i, c, acc, [] {});
    } else {
        a.in = o.in + rid * o.in_rs + (1 - P) * o.in_ss;
        hop_ahead<terms_ahead<SP, 1>(), SP, LK, 1, DAG>(a, PackedSrc<SP, true>{}, one, i, c, acc, [] {});
    }
    if constexpr (SP == SP_F64) {
        if (o.xpay) {
            double xv[24];
            if (o.xcanon) {
                const dbl2u_t *p = reinterpret_cast<const dbl2u_t *>(reinterpret_cast<const double *>(o.x) +
                                                                     rid * o.x_rs + site * 24);
#pragma unroll
                for (int k = 0; k < 12; k++) {
                    const dbl2u_t w = p[k];
                    xv[2 * k] = w.x;
                    xv[2 * k + 1] = w.y;
                }
            } else {
                SpinorIO<SP>::template load<true>(o.x + rid * o.x_rs + P * o.x_ss, o.g.cs, i, xv);
            }
#pragma unroll
            for (int k = 0; k < 24; k++) acc[0][k] = fmaT(o.coef, acc[0][k], xv[k]);
        }
    }
    if (!live) return;
    if (o.outcanon) {
        double d[24];
        stored_values<SP>(acc[0], d);
        dbl2u_t *p = reinterpret_cast<dbl2u_t *>(reinterpret_cast<double *>(o.out) + rid * o.out_rs + site * 24);
#pragma unroll
        for (int k = 0; k < 12; k++) p[k] = dbl2u_t{d[2 * k], d[2 * k + 1]};
    } else {
        SpinorIO<SP>::template store<true>(o.out + rid * o.out_rs + P * o.out_ss, o.g.cs, i, acc[0]);
    }
}

#define WD_OP_ONE(SP_, LK_, DAG_, CIN_)                                                           \
    hipLaunchKernelGGL((dslash_op_kernel<SP_, LK_, DAG_, CIN_>), grid, dim3(block), 0, s, o);     \
    return hipGetLastError();

#define WD_OP_LK(SP_, LK_)                                                                        \
    if (dag && o.incanon) { WD_OP_ONE(SP_, LK_, true, true) }                                     \
    if (dag) { WD_OP_ONE(SP_, LK_, true, false) }                                                 \
    if (o.incanon) { WD_OP_ONE(SP_, LK_, false, true) }                                           \
    WD_OP_ONE(SP_, LK_, false, false)

#define WD_OP_CASE(SP_, LK_)                                                                      \
    if (lk == LK_) { WD_OP_LK(SP_, LK_) }

}  // namespace wd
