// tune.hip -- launch-shape autotuner for the stencil sweeps of the solver and
// a stencil micro-benchmark.
//
// For each sweep the even-odd CG issues (plain D_oe, xpay+norm D_eo, plain
// D_oe^dag, fused CG-update D_eo^dag) in a given precision and RHS count, the
// tuner times every supported (block, RHS per lane, lanes per site, XCD
// remap) shape with HIP events on synthetic fields, re-runs each shape on
// identical inputs and rejects it unless its vectors and norm partials are
// bitwise identical to the reference shape, and keeps the fastest in the
// context.  Solves with wd_solver_params.tuned = 1 use the kept shapes.
#include <stdio.h>
#include <stdlib.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "wd_internal.h"

namespace wd {

namespace {

constexpr int kBlock = 256;

// deterministic pseudo-random fill in [-1, 1) (splitmix-style hash of the index)
template <int SP>
__global__ void __launch_bounds__(kBlock) k_fill(char *base, long long rs, int Vh, int cs, int nrhs,
                                                  unsigned seed)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    const int rid = blockIdx.y;
    if (i >= Vh || rid >= nrhs) return;
    double v[24];
    for (int k = 0; k < 24; k++) {
        unsigned long long z = ((unsigned long long)seed << 40) ^ ((unsigned long long)rid << 32) ^
                               ((unsigned long long)i * 24 + k);
        z += 0x9E3779B97F4A7C15ull;
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        z ^= z >> 31;
        v[k] = (double)(z >> 11) * (2.0 / 9007199254740992.0) - 1.0;
    }
    SpinorIO<SP>::store(base + rid * rs, cs, i, v);
}

__global__ void __launch_bounds__(kBlock) k_count_diff(const unsigned *a, const unsigned *b,
                                                        long long n, unsigned *count)
{
    const long long i = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (i < n && a[i] != b[i]) atomicAdd(count, 1u);
}

hipError_t fill(const Field &f, int Vh, int nrhs, unsigned seed, hipStream_t s)
{
    dim3 gr((Vh + kBlock - 1) / kBlock, nrhs);
    switch (f.sp) {
    case SP_F64: hipLaunchKernelGGL(k_fill<SP_F64>, gr, dim3(kBlock), 0, s, f.base, f.rs, Vh, f.cs, nrhs, seed); break;
    case SP_F32: hipLaunchKernelGGL(k_fill<SP_F32>, gr, dim3(kBlock), 0, s, f.base, f.rs, Vh, f.cs, nrhs, seed); break;
    case SP_F16: hipLaunchKernelGGL(k_fill<SP_F16>, gr, dim3(kBlock), 0, s, f.base, f.rs, Vh, f.cs, nrhs, seed); break;
    case SP_I16: hipLaunchKernelGGL(k_fill<SP_I16>, gr, dim3(kBlock), 0, s, f.base, f.rs, Vh, f.cs, nrhs, seed); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

__global__ void __launch_bounds__(kBlock) k_fill_bytes(unsigned *p, long long n, unsigned v)
{
    const long long i = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) p[i] = v * 0x01010101u;
}

hipError_t fill_bytes(void *p, size_t bytes, unsigned v, hipStream_t s)
{
    const long long n = (long long)(bytes / 4);
    if (n > 0)
        hipLaunchKernelGGL(k_fill_bytes, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s,
                           (unsigned *)p, n, v & 0xffu);
    return hipGetLastError();
}

std::string sweep_key(int sp, int lk, int dag, int epi)
{
    char b[64];
    snprintf(b, sizeof(b), "%d/%d/%d/%d", sp, lk, dag, epi);
    return b;
}

}  // namespace

const TuneCfg *tuned_cfg(const wd_ctx *c, const Sweep &sw)
{
    auto it = c->tuned.find(sweep_key(sw.sp, sw.lk, sw.dag, sw.epi));
    if (it == c->tuned.end() && sw.dag && sw.epi == EPI_XPAY)
        // H^dag with the xpay epilogue (the second factor of M^dag M in a
        // full-lattice solve) is not one of the four sweeps the tuner times: it
        // takes the shape tuned for D_eo^dag with the CG update, the same
        // stencil direction (every shape gives the same bits)
        it = c->tuned.find(sweep_key(sw.sp, sw.lk, 1, EPI_CGUPD));
    return it == c->tuned.end() ? nullptr : &it->second;
}

}  // namespace wd

using namespace wd;

#define HIPCHK(expr)                                                                               \
    do {                                                                                          \
        hipError_t e__ = (expr);                                                                  \
        if (e__ != hipSuccess)                                                                    \
            return set_error(WD_ERR_HIP, "%s: %s (%s:%d)", #expr, hipGetErrorString(e__), __FILE__, __LINE__); \
    } while (0)

static wd_status prec_decode(const wd_ctx *c, int prec, int *sp, int *lk, int *xp)
{
    return decode_prec(c, prec, sp, lk, xp);
}

struct TuneFields {
    Field in, out, x, r, r0, outref, rref;
    double *coef, *alpha, *partial, *pref;
    int *act;
    int pstride;
};

static wd_status tune_fields(wd_ctx *c, int sp, int nrhs, TuneFields *t)
{
    WD_TRY(alloc_field(c, "tn_in", sp, 1, nrhs, &t->in));
    WD_TRY(alloc_field(c, "tn_out", sp, 1, nrhs, &t->out));
    WD_TRY(alloc_field(c, "tn_x", sp, 1, nrhs, &t->x));
    WD_TRY(alloc_field(c, "tn_r", sp, 1, nrhs, &t->r));
    WD_TRY(alloc_field(c, "tn_r0", sp, 1, nrhs, &t->r0));
    WD_TRY(alloc_field(c, "tn_rref", sp, 1, nrhs, &t->rref));
    WD_TRY(alloc_field(c, "tn_outref", sp, 1, nrhs, &t->outref));
    const int Vh = (int)c->Vh;
    t->pstride = 2 * ngroups_of(Vh) + 1;
    std::vector<double> cf(nrhs), al(nrhs);
    std::vector<int> ids(nrhs);
    for (int j = 0; j < nrhs; j++) {
        cf[j] = -0.0243 - 0.0001 * j;  // about -kappa^2
        al[j] = 0.37 + 0.01 * j;
        ids[j] = j;
    }
    WD_TRY(upload_doubles(c, "tn_coef", cf.data(), nrhs, &t->coef));
    WD_TRY(upload_doubles(c, "tn_alpha", al.data(), nrhs, &t->alpha));
    WD_TRY(upload_ints(c, "tn_act", ids.data(), nrhs, &t->act));
    void *vp;
    WD_TRY(ws_get(c, "tn_partial", sizeof(double) * t->pstride * nrhs, &vp));
    t->partial = (double *)vp;
    WD_TRY(ws_get(c, "tn_pref", sizeof(double) * t->pstride * nrhs, &vp));
    t->pref = (double *)vp;
    hipStream_t s = c->stream;
    HIPCHK(fill(t->in, Vh, nrhs, 1, s));
    HIPCHK(fill(t->x, Vh, nrhs, 2, s));
    HIPCHK(fill(t->r0, Vh, nrhs, 4, s));
    HIPCHK(hipMemsetAsync(t->partial, 0, sizeof(double) * t->pstride * nrhs, s));
    return WD_OK;
}

// Bytes of the result fields of one sweep kind (for bitwise comparison).
static wd_status compare(wd_ctx *c, const char *a, const char *b, size_t bytes, unsigned *dcount,
                         unsigned *nd)
{
    hipStream_t s = c->stream;
    HIPCHK(hipMemsetAsync(dcount, 0, sizeof(unsigned), s));
    const long long n = (long long)(bytes / 4);
    if (n > 0)
        hipLaunchKernelGGL(k_count_diff, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s,
                           (const unsigned *)a, (const unsigned *)b, n, dcount);
    HIPCHK(hipGetLastError());
    HIPCHK(hipMemcpyAsync(nd, dcount, sizeof(unsigned), hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    return WD_OK;
}

// Tuning cache: a text file named by the environment variable
// WD_TUNE_CACHE, one line per tuned sweep:
//   Lx Ly Lz Lt nrhs sp lk dag epi block nr rl remap occ us [lnt]
// (lines without the occ field, from older files, read as occ = 0; without
// the trailing lnt field as lnt = 0)
static std::string cache_key(const wd_ctx *c, int nrhs, int sp, int lk, int dag, int epi)
{
    char b[128];
    snprintf(b, sizeof(b), "%d %d %d %d %d %d %d %d %d", c->dims[0], c->dims[1], c->dims[2], c->dims[3],
             nrhs, sp, lk, dag, epi);
    return b;
}

static bool cache_lookup(const char *path, const std::string &key, TuneCfg *cfg, double *us)
{
    FILE *f = fopen(path, "r");
    if (!f) return false;
    char line[256];
    bool found = false;
    while (fgets(line, sizeof(line), f)) {
        int d[9], b, nr, rl, rm, oc = 0, nt = 0;
        double t;
        double x[3];
        const int nf = sscanf(line, "%d %d %d %d %d %d %d %d %d %d %d %d %d %lf %lf %lf", &d[0], &d[1], &d[2],
                              &d[3], &d[4], &d[5], &d[6], &d[7], &d[8], &b, &nr, &rl, &rm, &x[0], &x[1], &x[2]);
        if (nf == 16) {
            oc = (int)x[0];
            t = x[1];
            nt = (int)x[2];
        } else if (nf == 15) {
            oc = (int)x[0];
            t = x[1];
        } else if (nf == 14) {
            t = x[0];
        } else {
            continue;
        }
        char k[128];
        snprintf(k, sizeof(k), "%d %d %d %d %d %d %d %d %d", d[0], d[1], d[2], d[3], d[4], d[5], d[6], d[7], d[8]);
        if (key == k) {  // the last matching line wins
            cfg->block = b;
            cfg->nr = nr;
            cfg->rl = rl;
            cfg->remap = rm;
            cfg->occ = oc;
            cfg->lnt = nt;
            *us = t;
            found = true;
        }
    }
    fclose(f);
    return found;
}

static void cache_store(const char *path, const std::string &key, const TuneCfg &cfg, double us)
{
    FILE *f = fopen(path, "a");
    if (!f) return;
    if (cfg.lnt)
        fprintf(f, "%s %d %d %d %d %d %.3f %d\n", key.c_str(), cfg.block, cfg.nr, cfg.rl, cfg.remap, cfg.occ, us,
                cfg.lnt);
    else
        fprintf(f, "%s %d %d %d %d %d %.3f\n", key.c_str(), cfg.block, cfg.nr, cfg.rl, cfg.remap, cfg.occ, us);
    fclose(f);
}

extern "C" wd_status wd_tune(wd_ctx *c, int nrhs, int prec, char *report, size_t len)
{
    if (!c) return set_error(WD_ERR_ARG, "NULL context");
    if (nrhs < 1 || nrhs > 64) return set_error(WD_ERR_ARG, "nrhs %d out of range 1..64", nrhs);
    if (!c->have_gauge) return set_error(WD_ERR_STATE, "no gauge field loaded");
    WD_HIP(hipSetDevice(c->device));
    int sp, lk, xp;
    WD_TRY(prec_decode(c, prec, &sp, &lk, &xp));
    const int Vh = (int)c->Vh;
    hipStream_t s = c->stream;
    TuneFields t;
    WD_TRY(tune_fields(c, sp, nrhs, &t));
    void *vp;
    WD_TRY(ws_get(c, "tn_count", sizeof(unsigned) * 4, &vp));
    unsigned *dcount = (unsigned *)vp;
    void *hp;
    WD_TRY(pinned_get(c, 1, 64, &hp));
    unsigned *nd = (unsigned *)hp;
    hipEvent_t e0, e1;
    WD_HIP(hipEventCreate(&e0));
    WD_HIP(hipEventCreate(&e1));
    const bool was_timing = c->timing;
    c->timing = false;

    std::vector<TuneCfg> cands;
    const int nrs[4] = {1, 2, 3, 4}, rls[3] = {1, 2, 4}, blocks[3] = {64, 128, 256};
    for (int rl : rls)
        for (int nr : nrs)
            for (int b : blocks)
                for (int rm = 0; rm < kTileOrders; rm++) {
                    if (!dslash_shape_supported(sp, lk, nr, rl)) continue;
                    if (rm >= 2 && !slab_order_ok(c->g, b / rl, rm)) continue;
                    if (nr * rl > 2 * nrhs && !(nr == 1 && rl == 1)) continue;  // mostly idle lanes
                    TuneCfg q;
                    q.block = b;
                    q.nr = nr;
                    q.rl = rl;
                    q.remap = rm;
                    cands.push_back(q);
                }
    // the LDS-staged t-walking kernel: 256 threads, one lane per site, 1 or 2
    // RHS per lane, 4, 8 or 16 t-planes per work-group
    for (int nr = 1; nr <= 2; nr++)
        for (int rm = kLdsOrder0; rm < kLdsOrder0 + kLdsOrders; rm++) {
            if (!lds_order_ok(c, sp, lk, nr, rm) || (nr > 2 * nrhs && nr != 1)) continue;
            TuneCfg q;
            q.block = 256;
            q.nr = nr;
            q.rl = 1;
            q.remap = rm;
            cands.push_back(q);
        }
    // the t-walking kernel with the t neighbours in registers: one lane per
    // site, tiles of the largest of 256, 128, 64 sites that divides a plane,
    // 1 to 3 RHS per lane, 4, 8 or 16 t-planes per work-group
    {
        const int S = c->g.Lxh * c->g.L[1];
        const int tb = S % 256 == 0 ? 256 : (S % 128 == 0 ? 128 : 64);
        for (int nr = 1; nr <= 3; nr++)
            for (int rm = kTwOrder0; rm < kTwOrder0 + kTwOrders; rm++) {
                if (!tw_order_ok(c, sp, lk, nr, 1, tb, rm) || (nr > 2 * nrhs && nr != 1)) continue;
                TuneCfg q;
                q.block = tb;
                q.nr = nr;
                q.rl = 1;
                q.remap = rm;
                cands.push_back(q);
            }
    }

    // (the solver's D_oe^dag sweep also finalizes alpha in extra work-groups:
    // timed here with them, on the partials and scalars of tn_fin)
    struct Kind { int P, dag, epi; const char *name; bool fin; };
    const Kind kinds[4] = {{1, 0, EPI_PLAIN, "D_oe", false}, {0, 0, EPI_XPAY, "xpay D_eo +norm", false},
                           {1, 1, EPI_PLAIN, "D_oe^dag", true}, {0, 1, EPI_CGUPD, "cg-update D_eo^dag", false}};
    WD_TRY(ws_get(c, "tn_fin", sizeof(double) * 3 * nrhs, &vp));
    double *fin = (double *)vp;
    HIPCHK(fill_bytes(fin, sizeof(double) * 3 * nrhs, 0x3Fu, s));  // finite positive doubles
    const size_t sb = (size_t)t.in.rs;  // bytes per RHS of a spinor field (padded)
    std::string rep;
    wd_status st = WD_OK;
    const char *cache = getenv("WD_TUNE_CACHE");
    // WD_TUNE_VERBOSE=1: every timed candidate on stderr
    const char *vb = getenv("WD_TUNE_VERBOSE");
    const bool verbose = vb && vb[0] == '1';
    for (const Kind &k : kinds) {
        Sweep sw;
        sw.sp = sp; sw.lk = lk; sw.dag = k.dag; sw.epi = k.epi; sw.P = k.P;
        sw.in = t.in; sw.out = t.out; sw.x = t.x; sw.r = t.r;
        sw.coef = t.coef; sw.alpha = t.alpha; sw.active = t.act; sw.nact = nrhs;
        sw.partial = (k.epi == EPI_PLAIN) ? nullptr : t.partial;
        sw.pstride = t.pstride;
        if (k.fin) {
            sw.fin_partial = t.pref;
            sw.fin_nw = ngroups_of(Vh);
            sw.fin_pstride = t.pstride;
            sw.fin_rr = fin;
            sw.fin_alpha = fin + nrhs;
            sw.fin_out = fin + 2 * nrhs;
        }

        // Runs list[0] (the reference shape) and then every other entry on
        // identical inputs, with every output poisoned first so that a shape
        // that skips sites cannot pass on stale results; a shape whose vectors
        // or norm partials differ in any bit from the reference is rejected
        // (ok[q] = false).  The accepted ones are timed (best of 3 batches of
        // 4 launches).  With occ_pass, the fastest shape of the list is then
        // retried with a cap of 2..kMaxOcc work-groups per CU.
        auto evaluate = [&](std::vector<TuneCfg> &list, bool occ_pass, std::vector<char> &ok,
                            std::vector<double> &us, TuneCfg &bestc, double &best) -> wd_status {
            best = 1e30;
            bestc = list[0];
            const size_t nfirst = list.size();
            bool nt_tried = false;
            for (size_t q = 0;; q++) {
                if (occ_pass && q == nfirst && best < 1e30 && !is_lds_order(bestc.remap))
                    for (int oc = 2; oc <= kMaxOcc; oc++) {
                        TuneCfg v = bestc;
                        v.occ = oc;
                        list.push_back(v);
                    }
                // then the best of all with its links loaded non-temporally
                if (occ_pass && q == list.size() && q > nfirst && !nt_tried && best < 1e30 &&
                    lnt_ok(sp, lk, bestc)) {
                    TuneCfg v = bestc;
                    v.lnt = 1;
                    list.push_back(v);
                    nt_tried = true;
                }
                if (q >= list.size()) break;
                ok.resize(list.size(), 0);
                us.resize(list.size(), 0.0);
                const TuneCfg cf = list[q];
                if (k.epi == EPI_CGUPD) {
                    HIPCHK(hipMemcpyAsync(t.r.base, t.r0.base, sb * nrhs, hipMemcpyDeviceToDevice, s));
                } else {
                    HIPCHK(fill(t.out, Vh, nrhs, 1000 + (unsigned)q, s));
                }
                // (the same poison every time: slots no shape writes stay equal)
                if (t.partial) HIPCHK(fill_bytes(t.partial, sizeof(double) * t.pstride * nrhs, 0xA5u, s));
                WD_TRY(run_sweep(c, sw, &cf));
                if (q == 0) {
                    HIPCHK(hipMemcpyAsync(t.outref.base, t.out.base, sb * nrhs, hipMemcpyDeviceToDevice, s));
                    HIPCHK(hipMemcpyAsync(t.rref.base, t.r.base, sb * nrhs, hipMemcpyDeviceToDevice, s));
                    HIPCHK(hipMemcpyAsync(t.pref, t.partial, sizeof(double) * t.pstride * nrhs,
                                          hipMemcpyDeviceToDevice, s));
                } else {
                    unsigned bad = 0;
                    if (k.epi == EPI_CGUPD) {
                        WD_TRY(compare(c, t.r.base, t.rref.base, sb * nrhs, dcount, nd));
                        bad += *nd;
                    } else {
                        WD_TRY(compare(c, t.out.base, t.outref.base, sb * nrhs, dcount, nd));
                        bad += *nd;
                    }
                    if (k.epi != EPI_PLAIN) {
                        WD_TRY(compare(c, (const char *)t.partial, (const char *)t.pref,
                                       sizeof(double) * t.pstride * nrhs, dcount, nd));
                        bad += *nd;
                    }
                    if (bad) continue;
                }
                ok[q] = 1;
                double tbest = 1e30;
                for (int rep3 = 0; rep3 < 3; rep3++) {
                    HIPCHK(hipEventRecord(e0, s));
                    for (int it = 0; it < 4; it++) WD_TRY(run_sweep(c, sw, &cf));
                    HIPCHK(hipEventRecord(e1, s));
                    HIPCHK(hipEventSynchronize(e1));
                    float ms = 0;
                    HIPCHK(hipEventElapsedTime(&ms, e0, e1));
                    tbest = std::min(tbest, (double)ms / 4);
                }
                us[q] = tbest * 1e3;
                if (verbose)
                    fprintf(stderr, "[wd tune] %s sp %d lk %d nrhs %d: block %d nr %d rl %d order %d cap %d nt %d: %.2f us\n",
                            k.name, sp, lk, nrhs, cf.block, cf.nr, cf.rl, cf.remap, cf.occ, cf.lnt, us[q]);
                if (tbest < best) {
                    best = tbest;
                    bestc = cf;
                }
            }
            return WD_OK;
        };
        auto rejected_of = [](const std::vector<char> &ok) {
            int r = 0;
            for (size_t q = 1; q < ok.size(); q++) r += ok[q] ? 0 : 1;
            return r;
        };
        auto report_line = [&](const TuneCfg &b, double us, double gbs, size_t ncand, int nrej, const char *src) {
            char line[320];
            snprintf(line, sizeof(line),
                     "%s;sp=%d;lk=%d;nrhs=%d;block=%d;nr=%d;rl=%d;remap=%d;occ=%d;lnt=%d;us=%.2f;GB/s=%.1f;"
                     "candidates=%zu;rejected=%d;source=%s\n",
                     k.name, sp, lk, nrhs, b.block, b.nr, b.rl, b.remap, b.occ, b.lnt, us, gbs, ncand, nrej, src);
            rep += line;
        };

        // A shape found in the cache is adopted only after it has given the
        // reference shape's results bit for bit on this lattice.
        if (cache && cache[0]) {
            TuneCfg cc;
            double us_cached = 0;
            if (cache_lookup(cache, cache_key(c, nrhs, sp, lk, k.dag, k.epi), &cc, &us_cached) &&
                dslash_shape_supported(sp, lk, cc.nr, cc.rl) && (cc.occ == 0 || (cc.occ >= 2 && cc.occ <= kMaxOcc)) &&
                (cc.lnt == 0 || (cc.lnt == 1 && lnt_ok(sp, lk, cc))) &&
                (is_lds_order(cc.remap)
                     ? (lds_order_ok(c, sp, lk, cc.nr, cc.remap) && cc.rl == 1 && cc.block == 256 && cc.occ == 0)
                 : is_tw_order(cc.remap)
                     ? tw_order_ok(c, sp, lk, cc.nr, cc.rl, cc.block, cc.remap)
                     : (cc.remap >= 0 && cc.remap < kTileOrders && cc.block >= 64 && cc.block <= 256 &&
                        (cc.block & 63) == 0 &&
                        (cc.remap < 2 || slab_order_ok(c->g, cc.block / cc.rl, cc.remap))))) {
                std::vector<TuneCfg> vl = {cands[0], cc};
                std::vector<char> ok;
                std::vector<double> us;
                TuneCfg bc;
                double bt;
                if ((st = evaluate(vl, false, ok, us, bc, bt)) != WD_OK) break;
                if (ok[1]) {
                    c->tuned[sweep_key(sp, lk, k.dag, k.epi)] = cc;
                    c->tune_gen++;
                    report_line(cc, us[1], sweep_bytes(c, sw) / (us[1] * 1e-6) / 1e9, 1, 0, "cache-verified");
                    continue;
                }
                // a cached shape that does not reproduce the reference is
                // discarded, and the sweep is tuned from scratch
                report_line(cc, us_cached, 0.0, 1, 1, "cache-rejected");
            }
        }
        std::vector<TuneCfg> list = cands;
        std::vector<char> ok;
        std::vector<double> us;
        TuneCfg bestc;
        double best;
        if ((st = evaluate(list, true, ok, us, bestc, best)) != WD_OK) break;
        c->tuned[sweep_key(sp, lk, k.dag, k.epi)] = bestc;
        c->tune_gen++;
        if (cache && cache[0]) cache_store(cache, cache_key(c, nrhs, sp, lk, k.dag, k.epi), bestc, best * 1e3);
        report_line(bestc, best * 1e3, sweep_bytes(c, sw) / (best * 1e-3) / 1e9, list.size(), rejected_of(ok),
                    "timed");
    }
    c->timing = was_timing;
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (st != WD_OK) return st;
    if (report && len) {
        if (rep.size() + 1 > len) return set_error(WD_ERR_ARG, "report needs %zu bytes", rep.size() + 1);
        memcpy(report, rep.c_str(), rep.size() + 1);
    }
    return WD_OK;
}

extern "C" wd_status wd_bench_dslash(wd_ctx *c, int nrhs, int prec, int epi, int iters, int tuned,
                                     double *ms, double *bytes)
{
    if (!c || !ms) return set_error(WD_ERR_ARG, "NULL argument");
    if (nrhs < 1 || nrhs > 64 || iters < 1 || epi < EPI_PLAIN || epi > EPI_CGUPD)
        return set_error(WD_ERR_ARG, "bad arguments");
    if (!c->have_gauge) return set_error(WD_ERR_STATE, "no gauge field loaded");
    WD_HIP(hipSetDevice(c->device));
    int sp, lk, xp;
    WD_TRY(prec_decode(c, prec, &sp, &lk, &xp));
    TuneFields t;
    WD_TRY(tune_fields(c, sp, nrhs, &t));
    hipStream_t s = c->stream;
    HIPCHK(hipMemcpyAsync(t.r.base, t.r0.base, (size_t)t.r.rs * nrhs, hipMemcpyDeviceToDevice, s));
    Sweep sw;
    // the CG update is timed as the solver runs it: on D_eo^dag (its fourth sweep)
    sw.sp = sp; sw.lk = lk; sw.dag = (epi == EPI_CGUPD) ? 1 : 0; sw.epi = epi; sw.P = (epi == EPI_PLAIN) ? 1 : 0;
    sw.in = t.in; sw.out = t.out; sw.x = t.x; sw.r = t.r;
    sw.coef = t.coef; sw.alpha = t.alpha; sw.active = t.act; sw.nact = nrhs;
    sw.partial = (epi == EPI_PLAIN) ? nullptr : t.partial;
    sw.pstride = t.pstride;
    const TuneCfg *cfg = tuned ? tuned_cfg(c, sw) : nullptr;
    // Back-to-back sweeps over one field would find much of it in the 256 MB
    // last-level cache: the timed sweeps rotate over nc copies of the links
    // and of every field, nc copies of the bytes a sweep moves reaching at
    // least 2 GiB, so that each sweep reads what the previous ones evicted.
    const double ws = sweep_bytes(c, sw);
    const int nc = (int)std::min(16.0, std::max(1.0, std::ceil(2.0 * 1073741824.0 / ws)));
    std::vector<Sweep> sws(nc, sw);
    const size_t lbytes = link_bytes(lk) * (size_t)8 * c->g.cs;
    for (int q = 1; q < nc; q++) {
        void *lp;
        WD_TRY(ws_get(c, "bd_links" + std::to_string(q), lbytes, &lp));
        HIPCHK(hipMemcpyAsync(lp, link_ptr(c, lk), lbytes, hipMemcpyDeviceToDevice, s));
        sws[q].links = (const char *)lp;
        Field *fs[4] = {&sws[q].in, &sws[q].out, &sws[q].x, &sws[q].r};
        const char *names[4] = {"bd_in", "bd_out", "bd_x", "bd_r"};
        for (int f = 0; f < 4; f++) {
            WD_TRY(alloc_field(c, names[f] + std::to_string(q), sp, 1, nrhs, fs[f]));
            HIPCHK(fill(*fs[f], (int)c->Vh, nrhs, 10 + f, s));
        }
    }
    WD_TRY(run_sweep(c, sw, cfg));  // warm-up
    hipEvent_t e0, e1;
    WD_HIP(hipEventCreate(&e0));
    WD_HIP(hipEventCreate(&e1));
    HIPCHK(hipEventRecord(e0, s));
    for (int it = 0; it < iters; it++) WD_TRY(run_sweep(c, sws[it % nc], cfg));
    HIPCHK(hipEventRecord(e1, s));
    HIPCHK(hipEventSynchronize(e1));
    float t_ms = 0;
    HIPCHK(hipEventElapsedTime(&t_ms, e0, e1));
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    // the copies go again (they are sized for this call only)
    for (int q = 1; q < nc; q++)
        for (const char *n : {"bd_links", "bd_in", "bd_out", "bd_x", "bd_r"}) {
            auto it = c->ws.find(n + std::to_string(q));
            if (it != c->ws.end()) {
                (void)hipFree(it->second.first);
                c->ws.erase(it);
            }
        }
    *ms = t_ms / iters;
    if (bytes) *bytes = ws;
    return WD_OK;
}
