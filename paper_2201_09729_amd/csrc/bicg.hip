// Site-local steps and scalar finishers of BiCGStab on the even-odd reduced operator
// Dhat (the alternative inner solver of dlma_solve).  One iteration is
//   v = Dhat p;            alpha = rho / (rh, v)
//   s = r - alpha v;       t = Dhat s;       omega = (t, s) / (t, t)
//   rho' = (rh, s) - omega (rh, t);          beta = (rho'/rho)(alpha/omega)
//   x += alpha p + omega s;  r = s - omega t;  p = r + beta (p - omega v)
// with (a, b) = sum conj(a_i) b_i over the even sites.  The operator applications
// are the solver's stencil kernels; everything here is a streaming pass over fields
// of the storage precision, in FP64 arithmetic, with deterministic two-stage sums.
// The shadow residual rh is a fixed seeded random field rather than the initial
// residual: a distillation source lives on one timeslice and one spin, and with
// rh = r_0 the scalar (rh, r) loses almost all of the spreading residual, which
// leaves the FP16 recursion to drift from the true residual.  Every right-hand
// side of a configuration reads the same field (its views have RHS stride 0), so
// the s step and K2 read it once per site rather than per RHS.
#include "kernels.h"

namespace dlma {

namespace {

struct Cd { double r, i; };
HD Cd cmulc(Cd a, Cd b) { return {a.r * b.r - a.i * b.i, a.r * b.i + a.i * b.r}; }
HD Cd cdivc(Cd a, Cd b) {
    const double d = b.r * b.r + b.i * b.i;
    return {(a.r * b.r + a.i * b.i) / d, (a.i * b.r - a.r * b.i) / d};
}
HD Cd ld2(const double2* p, int r) { const double2 v = p[r]; return {v.x, v.y}; }
HD bool finite2(Cd a) { return isfinite(a.r) && isfinite(a.i); }

// block sum of v written by thread 0 at part[idx]; every thread of the block calls it
__device__ __forceinline__ void bi_partial(double v, double* part, long idx) {
    __shared__ double lds[VEC_BS / 64];
    const double s = block_sum<VEC_BS>(v, lds);
    if (threadIdx.x == 0) part[idx] = s;
}

}  // namespace

// FP16 fields: the steps of one iteration in FP32 arithmetic on the raw words (128-bit
// loads and stores of the grouped layout, scales folded into the arithmetic).  FP32
// carries the 11-bit storage values and the FP64 scalars with margin; the partial
// sums are added in FP64.  Returns the NQ partial-sum contributions of the site.
HD void bv16_cplx(const uint32_t w[12], float n, float v[24]) {
#pragma unroll
    for (int c = 0; c < 12; ++c) {
        v[2 * c] = lo16(w[c]) * n;
        v[2 * c + 1] = hi16(w[c]) * n;
    }
}

template <int MODE> HD void bivec16(const BiVecJob<P16>& J, int r, uint32_t site, double& q0, double& q1) {
    const uint32_t Vh = (uint32_t)J.Vh, G16 = 16u * Vh, s16 = 16u * site, lo = 4u * site;
    uint32_t wa[12], wb[12], wc[12];
    float a[24], b[24], c[24];
    if (MODE == BV_SH) {  // s = r - alpha v, and (rh, s) of the stored s
        const F16Field R = f16_field(J.r, J.Vh, r), V = f16_field(J.v, J.Vh, r), S = f16_field(J.s, J.Vh, r);
        const F16Field RH = f16_field(J.rh, J.Vh, r);
        const float ar = (float)J.alpha[r].x, ai = (float)J.alpha[r].y;
        uint32_t wh[12];
        load_words<CP_NT>(R, s16, G16, wa);
        load_words<CP_NT>(V, s16, G16, wb);
        load_words(RH, s16, G16, wh);  // cached: every RHS reads this one field
        const float nr = wldf<CP_NT>(R.n, lo, 0), nv = wldf<CP_NT>(V.n, lo, 0), nh = wldf(RH.n, lo, 0);
        bv16_cplx(wa, nr, a);
        bv16_cplx(wb, nv, b);
#pragma unroll
        for (int i = 0; i < 12; ++i) {
            c[2 * i] = a[2 * i] - (ar * b[2 * i] - ai * b[2 * i + 1]);
            c[2 * i + 1] = a[2 * i + 1] - (ar * b[2 * i + 1] + ai * b[2 * i]);
        }
        float ms;
        (void)store16w(S, G16, site, c, wc, ms);
        float re, im;
        dot16(wh, wc, re, im);
        q0 = (double)re * ((double)nh * ms);
        q1 = (double)im * ((double)nh * ms);
    } else {  // BV_XRP: x += alpha p + omega s; r = s - omega t; p = r + beta (p - omega v); |r|^2
        const F16Field X = f16_field(J.x, J.Vh, r), Pp = f16_field(J.p, J.Vh, r), S = f16_field(J.s, J.Vh, r);
        const F16Field T = f16_field(J.t, J.Vh, r), R = f16_field(J.r, J.Vh, r), V = f16_field(J.v, J.Vh, r);
        const float alr = (float)J.alpha[r].x, ali = (float)J.alpha[r].y;
        const float omr = (float)J.omega[r].x, omi = (float)J.omega[r].y;
        const float ber = (float)J.beta[r].x, bei = (float)J.beta[r].y;
        // every load first (the stores could alias them as far as the compiler can tell)
        uint32_t wt[12], wv[12];
        load_words<CP_NT>(X, s16, G16, wa);
        load_words<CP_NT>(Pp, s16, G16, wb);
        load_words<CP_NT>(S, s16, G16, wc);
        load_words<CP_NT>(T, s16, G16, wt);
        load_words<CP_NT>(V, s16, G16, wv);
        const float nx = wldf<CP_NT>(X.n, lo, 0), np = wldf<CP_NT>(Pp.n, lo, 0), ns = wldf<CP_NT>(S.n, lo, 0);
        const float nt = wldf<CP_NT>(T.n, lo, 0), nv = wldf<CP_NT>(V.n, lo, 0);
        bv16_cplx(wa, nx, a);
        bv16_cplx(wb, np, b);
        bv16_cplx(wc, ns, c);
#pragma unroll
        for (int i = 0; i < 12; ++i) {  // x += alpha p + omega s
            const float pr = b[2 * i], pi = b[2 * i + 1], sr = c[2 * i], si = c[2 * i + 1];
            a[2 * i] += alr * pr - ali * pi + omr * sr - omi * si;
            a[2 * i + 1] += alr * pi + ali * pr + omr * si + omi * sr;
        }
        (void)store16(X, G16, site, a);
        bv16_cplx(wt, nt, a);
#pragma unroll
        for (int i = 0; i < 12; ++i) {  // r = s - omega t
            const float tr = a[2 * i], ti = a[2 * i + 1];
            c[2 * i] -= omr * tr - omi * ti;
            c[2 * i + 1] -= omr * ti + omi * tr;
        }
        q0 = (double)store16(R, G16, site, c);
        bv16_cplx(wv, nv, a);
#pragma unroll
        for (int i = 0; i < 12; ++i) {  // p = r + beta (p - omega v)
            const float dr = b[2 * i] - (omr * a[2 * i] - omi * a[2 * i + 1]);
            const float di = b[2 * i + 1] - (omr * a[2 * i + 1] + omi * a[2 * i]);
            b[2 * i] = c[2 * i] + ber * dr - bei * di;
            b[2 * i + 1] = c[2 * i + 1] + ber * di + bei * dr;
        }
        (void)store16(Pp, G16, site, b);
    }
}

// The FP64, FP32 and BF16 fields: half a spinor at a time, every load of it before its
// stores (which could alias them as far as the compiler can tell), FP64 arithmetic.
template <int P, int MODE> HD void bivec_planes(const BiVecJob<P>& J, int r, int cb, double& q0, double& q1) {
    using R = typename PT<P>::R;
    const int Vh = J.Vh;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        R a[12], b[12], c[12], d[12], f[12];
        if (MODE == BV_RR) {
            load_half_spinor<P, R>(J.rh, Vh, r, cb, h, a);
            load_half_spinor<P, R>(J.r, Vh, r, cb, h, c);
        } else if (MODE == BV_SH) {  // s = r - alpha v, and (rh, s) of the stored s
            const Cd al = ld2(J.alpha, r);
            load_half_spinor<P, R>(J.rh, Vh, r, cb, h, a);
            load_half_spinor<P, R>(J.r, Vh, r, cb, h, c);
            load_half_spinor<P, R>(J.v, Vh, r, cb, h, b);
#pragma unroll
            for (int i = 0; i < 12; i += 2) {
                const double br = b[i], bi = b[i + 1];
                c[i] = stored<P, R>((R)((double)c[i] - (al.r * br - al.i * bi)));
                c[i + 1] = stored<P, R>((R)((double)c[i + 1] - (al.r * bi + al.i * br)));
            }
            store_half_spinor<P, R>(J.s, Vh, r, cb, h, c);
        }
        if (MODE == BV_RR || MODE == BV_SH)
#pragma unroll
            for (int i = 0; i < 12; i += 2) {
                const double ar = a[i], ai = a[i + 1], br = c[i], bi = c[i + 1];
                q0 += ar * br + ai * bi;
                q1 += ar * bi - ai * br;
            }
        if (MODE == BV_XRP) {  // x += alpha p + omega s; r = s - omega t; p = r + beta (p - omega v); |r|^2
            const Cd al = ld2(J.alpha, r), om = ld2(J.omega, r), be = ld2(J.beta, r);
            load_half_spinor<P, R>(J.x, Vh, r, cb, h, a);
            load_half_spinor<P, R>(J.p, Vh, r, cb, h, b);
            load_half_spinor<P, R>(J.s, Vh, r, cb, h, c);
            load_half_spinor<P, R>(J.t, Vh, r, cb, h, d);
            load_half_spinor<P, R>(J.v, Vh, r, cb, h, f);
#pragma unroll
            for (int i = 0; i < 12; i += 2) {
                const double pr = b[i], pi = b[i + 1], sr = c[i], si = c[i + 1], tr = d[i], ti = d[i + 1], vr = f[i], vi = f[i + 1];
                a[i] = (R)((double)a[i] + al.r * pr - al.i * pi + om.r * sr - om.i * si);
                a[i + 1] = (R)((double)a[i + 1] + al.r * pi + al.i * pr + om.r * si + om.i * sr);
                c[i] = (R)(sr - (om.r * tr - om.i * ti));
                c[i + 1] = (R)(si - (om.r * ti + om.i * tr));
                const double rr = c[i], ri = c[i + 1], gr = pr - (om.r * vr - om.i * vi), gi = pi - (om.r * vi + om.i * vr);
                b[i] = (R)(rr + be.r * gr - be.i * gi);
                b[i + 1] = (R)(ri + be.r * gi + be.i * gr);
                q0 += rr * rr + ri * ri;
            }
            store_half_spinor<P, R>(J.x, Vh, r, cb, h, a);
            store_half_spinor<P, R>(J.r, Vh, r, cb, h, c);
            store_half_spinor<P, R>(J.p, Vh, r, cb, h, b);
        }
    }
}

template <int P, int MODE> __global__ void __launch_bounds__(VEC_BS) k_bivec(const BiVecJob<P>* jobs, int njob) {
    const int bid = blockIdx.x;
    int jb = 0;
    while (jb + 1 < njob && bid >= jobs[jb + 1].blk0) ++jb;
    const BiVecJob<P>& J = jobs[jb];
    const int lb = bid - J.blk0;
    const int r = lb / J.nsb;
    const int sb = lb - r * J.nsb;
    const int cb = sb * VEC_BS + (int)threadIdx.x;
    const bool act = rhs_active(J, r);  // uniform over the block
    constexpr int NQ = MODE == BV_XRP ? 1 : 2;
    double* part = MODE == BV_SH ? J.part_s : J.part;
    if (!act) {  // the whole block: zero partials, no block sums
        if ((int)threadIdx.x < NQ) part[((long)r * NQ + (int)threadIdx.x) * J.pstride + sb] = 0.0;
        return;
    }
    double q0 = 0, q1 = 0;
    if constexpr (P == P16 && MODE != BV_RR) {
        // first pass: beyond the reach of the outputs everything is zero and stays so
        constexpr int reach = MODE == BV_SH ? 3 : 5;
        const bool near = cb < J.Vh && in_reach(J.tdist, J.titer, J.T, r, J.tdist ? cb / J.vt : 0, reach);
        if (near) bivec16<MODE>(J, r, (uint32_t)cb, q0, q1);
    } else if constexpr (P == P16) {
        if (cb < J.Vh) {
            float a[24], b[24];
            load_spinor<P, float>(J.rh, J.Vh, r, cb, a);
            load_spinor<P, float>(J.r, J.Vh, r, cb, b);
            for (int i = 0; i < 12; ++i) {
                const double ar = a[2 * i], ai = a[2 * i + 1], br = b[2 * i], bi = b[2 * i + 1];
                q0 += ar * br + ai * bi;
                q1 += ar * bi - ai * br;
            }
        }
    } else {
        if (cb < J.Vh) bivec_planes<P, MODE>(J, r, cb, q0, q1);
    }
    bi_partial(q0, part, ((long)r * NQ + 0) * J.pstride + sb);
    if (NQ > 1) bi_partial(q1, part, ((long)r * NQ + 1) * J.pstride + sb);
}

template <int P> hipError_t launch_bivec(const BiVecJob<P>* j, int njob, int nblocks, int mode, hipStream_t s) {
    if (nblocks <= 0) return hipSuccess;
    switch (mode) {
    case BV_RR: hipLaunchKernelGGL((k_bivec<P, BV_RR>), dim3(nblocks), dim3(VEC_BS), 0, s, j, njob); break;
    case BV_SH: hipLaunchKernelGGL((k_bivec<P, BV_SH>), dim3(nblocks), dim3(VEC_BS), 0, s, j, njob); break;
    case BV_XRP: hipLaunchKernelGGL((k_bivec<P, BV_XRP>), dim3(nblocks), dim3(VEC_BS), 0, s, j, njob); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template hipError_t launch_bivec<P64>(const BiVecJob<P64>*, int, int, int, hipStream_t);
template hipError_t launch_bivec<P32>(const BiVecJob<P32>*, int, int, int, hipStream_t);
template hipError_t launch_bivec<P16>(const BiVecJob<P16>*, int, int, int, hipStream_t);
template hipError_t launch_bivec<PB16>(const BiVecJob<PB16>*, int, int, int, hipStream_t);

// One block per right-hand side: fixed-order sums of the quantities' partials, then
// the scalar update of the mode.  A right-hand side stops (inactive) when |r|^2
// reaches its target, at the iteration cap, on a non-finite value, or on a
// breakdown (a zero denominator); the defect-correction pass that runs the inner
// solve restarts from the true residual in every case.
// A chain of latencies (partials, sums, scalars): every quantity's partials are loaded
// together and one barrier serves all sums.  4.7 to 7.2 us, 20 us with 1300 partials, when each
// quantity had its own pass and barriers; now 3.9 to 6.5 us.
template <int mode> __global__ void __launch_bounds__(256) k_bifinish(const BiFinJob* jobs, int njob) {
    const int bid = blockIdx.x;
    int jb = 0;
    while (jb + 1 < njob && bid >= jobs[jb + 1].rhs0) ++jb;
    const BiFinJob& J = jobs[jb];
    const int r = bid - J.rhs0;
    if (r >= J.nrhs) return;  // uniform over the block
    constexpr int NQ = (mode == BF_ALPHA || mode == BF_INIT) ? 2 : (mode == BF_OMBETA ? 5 : 1);
    constexpr int NS = mode == BF_OMBETA ? 2 : 0;  // (rh, s) from the s step's own partials
    const int np = (mode == BF_ALPHA || mode == BF_OMBETA) ? J.nparth : J.npart;
    double q[7] = {0, 0, 0, 0, 0, 0, 0};
    const double* pp = J.part + (size_t)r * NQ * np;
#pragma unroll 4
    for (int i = threadIdx.x; i < np; i += 256)
#pragma unroll
        for (int k = 0; k < NQ; ++k) q[k] += pp[(size_t)k * np + i];
    if (NS > 0) {
        const double* ps = J.part_s + (size_t)r * 2 * J.npart;
#pragma unroll 4
        for (int i = threadIdx.x; i < J.npart; i += 256)
#pragma unroll
            for (int k = 0; k < NS; ++k) q[5 + k] += ps[(size_t)k * J.npart + i];
    }
    __shared__ double lds[7][4];
    auto wave = [&](int k) {
        double v = q[k];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        if ((threadIdx.x & 63) == 0) lds[k][threadIdx.x >> 6] = v;
    };
#pragma unroll
    for (int k = 0; k < NQ; ++k) wave(k);
#pragma unroll
    for (int k = 0; k < NS; ++k) wave(5 + k);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 7; ++k)
        if (k < NQ || (k >= 5 && k < 5 + NS)) q[k] = ((lds[k][0] + lds[k][1]) + lds[k][2]) + lds[k][3];
    if (threadIdx.x != 0) return;
    const Cd one = {1.0, 0.0}, zero = {0.0, 0.0};
    auto st = [](double2* a, int i, Cd v) { a[i] = make_double2(v.r, v.i); };
    if (mode == BF_INIT) {  // start of an inner solve (after the CG-state init): rho = (rh, r)
        const Cd rho = {q[0], q[1]};
        st(J.rho, r, rho);
        st(J.alpha, r, one);
        st(J.omega, r, one);
        st(J.beta, r, zero);
        if (J.active[r] && (!finite2(rho) || (rho.r == 0.0 && rho.i == 0.0))) J.active[r] = 0;
        return;
    }
    if (!J.active[r]) return;
    if (mode == BF_ALPHA) {
        const Cd d = {q[0], q[1]};
        if (!finite2(d) || (d.r == 0.0 && d.i == 0.0)) {
            st(J.alpha, r, zero);
            J.active[r] = 0;
        } else {
            st(J.alpha, r, cdivc(ld2(J.rho, r), d));
        }
    } else if (mode == BF_OMBETA) {
        // omega = (t, s) / |t|^2; rho' = (rh, s) - omega (rh, t), both on the stored s and t, is
        // (rh, s - omega t) for the r = s - omega t that the merged update forms from them
        const Cd ts = {q[0], q[1]}, rt = {q[3], q[4]}, rs = {q[5], q[6]};
        const Cd om = (finite2(ts) && q[2] > 0.0 && isfinite(q[2])) ? Cd{ts.r / q[2], ts.i / q[2]} : zero;
        st(J.omega, r, om);
        const Cd ort = cmulc(om, rt);
        const Cd rho1 = {rs.r - ort.r, rs.i - ort.i};
        const Cd rho = ld2(J.rho, r), al = ld2(J.alpha, r);
        const bool brk = (om.r == 0.0 && om.i == 0.0) || (rho.r == 0.0 && rho.i == 0.0) || !finite2(rho1) ||
                         (rho1.r == 0.0 && rho1.i == 0.0);
        // on a breakdown the update still runs (with beta = 0) and BF_CONV stops the right-hand side
        st(J.beta, r, brk ? zero : cmulc(cdivc(rho1, rho), cdivc(al, om)));
        st(J.rho, r, brk ? zero : rho1);
    } else {  // BF_CONV
        const double rr = q[0];
        J.rr[r] = rr;
        const int it = J.iters[r] + 1;
        J.iters[r] = it;
        const Cd rho = ld2(J.rho, r);  // zero after a breakdown
        if (!isfinite(rr) || rr <= J.tol2[r] || it >= J.maxit || (rho.r == 0.0 && rho.i == 0.0)) J.active[r] = 0;
    }
}

hipError_t launch_bifinish(const BiFinJob* j, int njob, int nblocks, int mode, hipStream_t s) {
    if (nblocks <= 0) return hipSuccess;
    const dim3 g(nblocks), b(256);
    switch (mode) {
    case BF_INIT: hipLaunchKernelGGL(k_bifinish<BF_INIT>, g, b, 0, s, j, njob); break;
    case BF_ALPHA: hipLaunchKernelGGL(k_bifinish<BF_ALPHA>, g, b, 0, s, j, njob); break;
    case BF_OMBETA: hipLaunchKernelGGL(k_bifinish<BF_OMBETA>, g, b, 0, s, j, njob); break;
    case BF_CONV: hipLaunchKernelGGL(k_bifinish<BF_CONV>, g, b, 0, s, j, njob); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace dlma
