// D and D^dag of the full FP64 operator on fields in the canonical order: one pass over the
// fields (a conversion to the even-odd planes and back took 0.58 + 0.55 ms of 3.15 ms for
// D^dag on 24^3 x 48 with 12 right-hand sides, and 20 of 44 us on 4^4).
//
// Block order of both kernels: an XCD owns a range of timeslices (and of z, where T does
// not divide by 8), walks strips of a plane outermost, then z, then its timeslices, so the
// +-t and +-z neighbours of a strip stay in its L2; the right-hand sides of a place come
// together and share its links.
#include <algorithm>
#include <numeric>
#include "kernels.h"

namespace dlma {

namespace {

typedef double D2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ double quad_swap(double v, int ctl) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    uint32_t lo = (uint32_t)b, hi = (uint32_t)(b >> 32);
    if (ctl == 1) {  // lanes l ^ 1
        lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)lo, 0xB1, 0xf, 0xf, true);
        hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)hi, 0xB1, 0xf, 0xf, true);
    } else {  // lanes l ^ 2
        lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)lo, 0x4E, 0xf, 0xf, true);
        hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)hi, 0x4E, 0xf, 0xf, true);
    }
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ double2 quad_swap(double2 v, int ctl) { return make_double2(quad_swap(v.x, ctl), quad_swap(v.y, ctl)); }

// a += s b and a += s i b, s real
__device__ __forceinline__ void add_re(double2& a, double s, double2 b) { a.x = fma(s, b.x, a.x); a.y = fma(s, b.y, a.y); }
__device__ __forceinline__ void add_im(double2& a, double s, double2 b) { a.x = fma(-s, b.y, a.x); a.y = fma(s, b.x, a.y); }
__device__ __forceinline__ void add_mul(double2& a, double2 m, double2 b) {
    a.x = fma(m.x, b.x, a.x);
    a.x = fma(-m.y, b.y, a.x);
    a.y = fma(m.x, b.y, a.y);
    a.y = fma(m.y, b.x, a.y);
}

// Four lanes take one output site, lane (f, p) = (l / 2, l % 2): f = 0 the forward and
// f = 1 the backward neighbour of each direction, p the two components of the
// half-spinor.  With h_p = psi_p + sigma_f g_{p,c} psi_c at the neighbour (sigma = -1
// forward, +1 backward, c = 2 + p or 3 - p the column of g_mu's entry in row p) and
// r_p = U' h_p, the site's sum is, over f, mu,
//   row p: r_p,   row c: sigma_f g_{c,p} r_p,
// gathered per lane (lo: row 2 + p, sw: row 3 - p) and exchanged among the four lanes
// once at the end; lane l then holds row l, which is also its row of the clover term.  So
// every spin of a neighbour is loaded once, and short calls have four waves per 64 sites.
// Bound: latency, 4^4 in 24 us per call of which the kernel is 6; at large sizes the
// scattered loads (41 pieces of 64 bytes per load instruction against 24 below).
__global__ void __launch_bounds__(256) k_dirac(DiracArgs a) {
    // wave -> (super-group of right-hand sides, strip of rows, z, t, sites, group)
    const Geo& g = a.g;
    const int xcd = (int)(blockIdx.x & 7), ti = xcd % a.nT, zi = xcd / a.nT, nZ = 8 / a.nT;
    const int t0 = ti * g.T / a.nT, nt = (ti + 1) * g.T / a.nT - t0;
    const int z0 = zi * g.Z / nZ, nz = (zi + 1) * g.Z / nZ - z0;
    long w = (long)(blockIdx.x >> 3) * 4 + (threadIdx.x >> 6);
    const int grp = (int)(w % a.ng); w /= a.ng;
    const int ch = (int)(w % a.nch); w /= a.nch;
    if (nt == 0 || nz == 0) return;
    const int t = t0 + (int)(w % nt); w /= nt;
    const int z = z0 + (int)(w % nz); w /= nz;
    const int strip = (int)(w % a.nstrip); w /= a.nstrip;
    const int r = (int)w * a.ng + grp;
    if (r >= a.nrhs) return;
    const int lane = (int)threadIdx.x & 63, l = lane & 3, p = l & 1;
    const bool bw = l >= 2;
    const int rows = min(a.R, g.Y - strip * a.R), ns = rows * g.X;
    int i = ch * 16 + (lane >> 2);
    const bool on = i < ns;
    if (!on) i = ns - 1;
    const int y = strip * a.R + (int)((uint32_t)i / (uint32_t)g.X), x = i - (y - strip * a.R) * g.X;
    const int par = (t + z + y + x) & 1;
    const int cb = ((t * g.Z + z) * g.Y + y) * g.Xh + (x >> 1);
    const double sg = bw ? a.sg : -a.sg, sp = p ? sg : -sg;  // sigma_f, and with the sign of rows p in g_2, g_3
    const double cj = bw ? -1.0 : 1.0;
    const long rs = (long)r * 24 * g.Vh;

    double2 up[3], lo[3], sw[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) up[c] = lo[c] = sw[c] = make_double2(0.0, 0.0);
    const uint32_t sa = bw ? (uint32_t)g.Vh : 3u * (uint32_t)g.Vh, sb = bw ? 3u * (uint32_t)g.Vh : (uint32_t)g.Vh;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {

        // this lane's neighbour
        int xt = t, xz = z, xy = y, xx = x;
        const int d = bw ? -1 : 1;
        auto wrap = [](int v, int n) { return v < 0 ? n - 1 : (v == n ? 0 : v); };
        if (mu == 0) xt = wrap(t + d, g.T);
        if (mu == 1) xx = wrap(x + d, g.X);
        if (mu == 2) xy = wrap(y + d, g.Y);
        if (mu == 3) xz = wrap(z + d, g.Z);
        const int row = (xt * g.Z + xz) * g.Y + xy;
        const long ns0 = (long)row * g.X + xx;
        // its link: U_mu(x), or U_mu(x - mu) at the neighbour
        const int lcb = bw ? row * g.Xh + (xx >> 1) : cb, lpar = bw ? 1 - par : par;
        const double2* U = a.U + (long)(lpar * 4 + mu) * 9 * g.Vh + lcb;
        double2 m[3][3];
#pragma unroll
        for (int b = 0; b < 3; ++b)
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                m[b][e] = U[b * sa + e * sb];
                m[b][e].y *= cj;
            }
        const int c = (mu == 0 || mu == 3) ? 2 + p : 3 - p;
        const double2* f0 = a.in + rs + (ns0 * 4 + p) * 3;
        const double2* f1 = a.in + rs + (ns0 * 4 + c) * 3;
        double2 h[3];
#pragma unroll
        for (int e = 0; e < 3; ++e) {
            h[e] = f0[e];
            const double2 k = f1[e];
            if (mu == 0) add_re(h[e], -sg, k);
            if (mu == 1) add_im(h[e], -sg, k);
            if (mu == 2) add_re(h[e], sp, k);
            if (mu == 3) add_im(h[e], sp, k);
        }
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            double2 r = make_double2(0.0, 0.0);
#pragma unroll
            for (int e = 0; e < 3; ++e) add_mul(r, m[b][e], h[e]);
            up[b].x += r.x;
            up[b].y += r.y;
            if (mu == 0) add_re(lo[b], -sg, r);
            if (mu == 1) add_im(sw[b], sg, r);
            if (mu == 2) add_re(sw[b], sp, r);
            if (mu == 3) add_im(lo[b], -sp, r);
        }
    }
    // clover: lane l holds row l = spin p of chirality bw; entries of the packed Hermitian
    // block, diagonal pairs first, then the lower triangle
    const double2* C = (par ? a.C1 : a.C0) + ((long)(bw ? 1 : 0) * 18) * g.Vh + cb;
    const uint32_t Vh = (uint32_t)g.Vh;
    auto tri = [](int i, int j) { return 3 + i * (i - 1) / 2 + j; };  // i > j
    double2 own[3], crs[3][3];  // own block (1,0), (2,0), (2,1); crossing: rows own, columns the other spin's
    double dg[3];
    {
        const double2 d1 = C[(p ? 1u : 0u) * Vh], d2 = C[(p ? 2u : 1u) * Vh];
        dg[0] = p ? d1.y : d1.x;
        dg[1] = p ? d2.x : d1.y;
        dg[2] = p ? d2.y : d2.x;
    }
    own[0] = C[(uint32_t)(p ? tri(4, 3) : tri(1, 0)) * Vh];
    own[1] = C[(uint32_t)(p ? tri(5, 3) : tri(2, 0)) * Vh];
    own[2] = C[(uint32_t)(p ? tri(5, 4) : tri(2, 1)) * Vh];
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int e = 0; e < 3; ++e) {
            crs[b][e] = C[(uint32_t)(p ? tri(3 + b, e) : tri(3 + e, b)) * Vh];
            crs[b][e].y *= p ? 1.0 : -1.0;
        }
    const long me = rs + (((long)((t * g.Z + z) * g.Y + y) * g.X + x) * 4 + l) * 3;
    double2 v[3], q[3], s[3];
#pragma unroll
    for (int e = 0; e < 3; ++e) v[e] = a.in[me + e];
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        q[e] = quad_swap(v[e], 1);
        const double2 k = quad_swap(sw[e], 1);
        const double2 low = make_double2(lo[e].x + k.x, lo[e].y + k.y);
        const double2 give = bw ? up[e] : low, keep = bw ? low : up[e];
        const double2 got = quad_swap(give, 2);
        s[e] = make_double2(-0.5 * (keep.x + got.x), -0.5 * (keep.y + got.y));
    }
    auto conj = [](double2 z) { return make_double2(z.x, -z.y); };
    add_mul(s[1], own[0], v[0]);
    add_mul(s[0], conj(own[0]), v[1]);
    add_mul(s[2], own[1], v[0]);
    add_mul(s[0], conj(own[1]), v[2]);
    add_mul(s[2], own[2], v[1]);
    add_mul(s[1], conj(own[2]), v[2]);
#pragma unroll
    for (int b = 0; b < 3; ++b) {
#pragma unroll
        for (int e = 0; e < 3; ++e) add_mul(s[b], crs[b][e], q[e]);
        add_re(s[b], dg[b], v[b]);  // the largest term last: fewest roundings at its size
        if (on) a.out[me + b] = s[b];
    }
}

// One lane per site, a wave 64 consecutive sites of a (t, z) plane and one right-hand side.
// Each neighbour set (and the wave's own sites) is read as contiguous 1 KB pieces, passes
// through the wave's LDS (sites 13 numbers apart: few bank conflicts), and the next one is
// on its way while this one is worked on; the own sites come last, with the clover term.
// Bound: the vector memory path (texture address unit 0.97 busy, 228 loads and stores per wave, 3.8
// times the compulsory reads from the memory side: 5.9 TB/s in all), at two waves per SIMD (236
// registers; three waves spill and take twice as long).  24^3 x 48, D^dag, per call: one right-hand side 462 to
// 267 us, 12 3151 to 1680 us (3.8 GB of fields, links and clover once: 2.3 TB/s).
constexpr int PAD = 13;

// the same on native vectors
__device__ __forceinline__ void add_re(D2& a, double s, D2 b) { a.x = fma(s, b.x, a.x); a.y = fma(s, b.y, a.y); }
__device__ __forceinline__ void add_im(D2& a, double s, D2 b) { a.x = fma(-s, b.y, a.x); a.y = fma(s, b.x, a.y); }
__device__ __forceinline__ void add_mul(D2& a, double mx, double my, D2 b) {
    a.x = fma(mx, b.x, a.x);
    a.x = fma(-my, b.y, a.x);
    a.y = fma(mx, b.y, a.y);
    a.y = fma(my, b.x, a.y);
}

template <int D>  // direction 2 mu + backward; ps: psi of the neighbour, acc: the sum over directions
__device__ __forceinline__ void hop_site(const D2* ps, const D2 (&m)[9], double sgd, D2 (&acc)[12]) {
    constexpr int mu = D >> 1;
    const double sg = (D & 1) ? sgd : -sgd;
    // row p, column c of g_mu; the entry of row c is its conjugate
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        constexpr bool straight = mu == 0 || mu == 3;
        const int c = straight ? 2 + p : 3 - p;
        D2 h[3];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < 3; ++e) {
            h[e] = ps[p * 3 + e];
            const D2 k = ps[c * 3 + e];
            if (mu == 0) add_re(h[e], -sg, k);
            if (mu == 1) add_im(h[e], -sg, k);
            if (mu == 2) add_re(h[e], p ? sg : -sg, k);
            if (mu == 3) add_im(h[e], p ? sg : -sg, k);
        }
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            D2 r = {0.0, 0.0};
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                const D2 u = m[(D & 1) ? e * 3 + b : b * 3 + e];
                add_mul(r, u.x, (D & 1) ? -u.y : u.y, h[e]);
            }
            acc[p * 3 + b] += r;
            if (mu == 0) add_re(acc[c * 3 + b], -sg, r);
            if (mu == 1) add_im(acc[c * 3 + b], sg, r);
            if (mu == 2) add_re(acc[c * 3 + b], p ? sg : -sg, r);
            if (mu == 3) add_im(acc[c * 3 + b], p ? -sg : sg, r);
        }
    }
}

struct SiteWave {  // a wave's place
    const double2* in;    // its right-hand side
    D2* buf;
    int t, z, plane, e0, e1, lane;
    int pos[3];           // place of piece k in the buffer: pos[k % 3] + k / 3 * 16 PAD
    uint32_t xlo, xhi;    // pieces whose site has x = 0, x = X - 1
    int x, y, par, cb;    // this lane's site
};
__device__ __forceinline__ int wrap1(int v, int n) { return v < 0 ? n - 1 : (v == n ? 0 : v); }

// p[i] by a 32-bit byte offset from a uniform address
__device__ __forceinline__ D2 at32(const double2* p, uint32_t i) { return *(const D2*)((const char*)p + (size_t)(i * 16u)); }

// Sites of direction D (8: its own): 768 numbers e = 64 k + lane, site e / 12 of the wave,
// clamped to its last
template <int D> __device__ __forceinline__ void fetch(const SiteWave& w, const Geo& g, D2 (&st)[12]) {
    constexpr int s = (D & 1) ? -1 : 1;
    const int t = D >> 1 == 0 ? wrap1(w.t + s, g.T) : w.t, z = D >> 1 == 3 ? wrap1(w.z + s, g.Z) : w.z;
    const double2* f = w.in + (long)(t * g.Z + z) * w.plane * 12;
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        int e = w.e0 + min(64 * k + w.lane, w.e1);
        if (D == 2) e += (w.xhi >> k & 1) ? 12 - 12 * g.X : 12;
        if (D == 3) e += (w.xlo >> k & 1) ? 12 * g.X - 12 : -12;
        if (D == 4) { e += 12 * g.X; e = e >= 12 * w.plane ? e - 12 * w.plane : e; }
        if (D == 5) { e -= 12 * g.X; e = e < 0 ? e + 12 * w.plane : e; }
        st[k] = at32(f, (uint32_t)e);
    }
}
__device__ __forceinline__ void place(const SiteWave& w, const D2 (&st)[12]) {
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int k = 0; k < 12; ++k) w.buf[w.pos[k % 3] + k / 3 * 16 * PAD] = st[k];
    __builtin_amdgcn_wave_barrier();
}

// the link of direction D
template <int D> __device__ __forceinline__ void link(const SiteWave& w, const DiracArgs& a, D2 (&m)[9]) {
    const Geo& g = a.g;
    int t = w.t, z = w.z, y = w.y, x = w.x;
    if (D == 1) t = wrap1(t - 1, g.T);
    if (D == 3) x = wrap1(x - 1, g.X);
    if (D == 5) y = wrap1(y - 1, g.Y);
    if (D == 7) z = wrap1(z - 1, g.Z);
    const int cb = (D & 1) ? ((t * g.Z + z) * g.Y + y) * g.Xh + (x >> 1) : w.cb, par = (D & 1) ? 1 - w.par : w.par;
    const uint32_t o = (uint32_t)(par * 36) * (uint32_t)g.Vh + (uint32_t)cb;
#pragma unroll
    for (int k = 0; k < 9; ++k) m[k] = at32(a.U + (size_t)((D >> 1) * 9 + k) * g.Vh, o);
}

template <int D>
__device__ __forceinline__ void hop_step(const SiteWave& w, const DiracArgs& a, D2 (&st)[12], D2 (&acc)[12]) {
    __builtin_amdgcn_sched_barrier(0);
    place(w, st);
    // the link first, then the next neighbours: loads come back in order
    D2 m[9];
    link<D>(w, a, m);
    fetch<D + 1>(w, a.g, st);  // (8: its own sites)
    __builtin_amdgcn_sched_barrier(0);
    hop_site<D>(w.buf + w.lane * PAD, m, a.sg, acc);
}

__global__ void __launch_bounds__(256, 2) k_dirac_sites(DiracArgs a) {
    const Geo& g = a.g;
    const int xcd = (int)(blockIdx.x & 7), ti = xcd % a.nT, zi = xcd / a.nT, nZ = 8 / a.nT;
    const int t0 = ti * g.T / a.nT, nt = (ti + 1) * g.T / a.nT - t0;
    const int z0 = zi * g.Z / nZ, nz = (zi + 1) * g.Z / nZ - z0;
    if (nt == 0 || nz == 0) return;
    // wave -> (super-group of right-hand sides, strip of the plane, z, t, 64 sites, right-hand side)
    const int wv = wave_uniform((int)(threadIdx.x >> 6));
    uint32_t i = (blockIdx.x >> 3) * 4 + (uint32_t)wv;
    const int grp = (int)(i % (uint32_t)a.ng); i /= (uint32_t)a.ng;
    const int ch = (int)(i % (uint32_t)a.nch); i /= (uint32_t)a.nch;
    SiteWave w;
    w.t = t0 + (int)(i % (uint32_t)nt); i /= (uint32_t)nt;
    w.z = z0 + (int)(i % (uint32_t)nz); i /= (uint32_t)nz;
    const int strip = (int)(i % (uint32_t)a.nstrip); i /= (uint32_t)a.nstrip;
    const int r = (int)i * a.ng + grp;
    if (r >= a.nrhs) return;
    w.plane = g.Y * g.X;
    const int s0 = (strip * a.nch + ch) * 64;
    if (s0 >= w.plane) return;
    __shared__ D2 lds[4][64 * PAD];
    w.lane = (int)threadIdx.x & 63;
    w.buf = lds[wv];
    const long rs = (long)r * 24 * g.Vh;
    w.in = a.in + rs;
    const int ns = min(64, w.plane - s0);
    w.e0 = 12 * s0;
    w.e1 = 12 * ns - 1;
#pragma unroll
    for (int k = 0; k < 3; ++k) w.pos[k] = 64 * k + w.lane + (64 * k + w.lane) / 12;
    w.xlo = w.xhi = 0;
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        const uint32_t x = (uint32_t)(w.e0 + min(64 * k + w.lane, w.e1)) / 12u % (uint32_t)g.X;
        w.xlo |= x == 0 ? 1u << k : 0u;
        w.xhi |= x == (uint32_t)g.X - 1 ? 1u << k : 0u;
    }
    const int site = s0 + min(w.lane, ns - 1);
    w.y = (int)((uint32_t)site / (uint32_t)g.X);
    w.x = site - w.y * g.X;
    w.par = (w.t + w.z + w.y + w.x) & 1;
    w.cb = ((w.t * g.Z + w.z) * g.Y + w.y) * g.Xh + (w.x >> 1);

    D2 st[12];
    D2 acc[12];
#pragma unroll
    for (int e = 0; e < 12; ++e) acc[e] = (D2){0.0, 0.0};
    fetch<0>(w, g, st);
    hop_step<0>(w, a, st, acc);
    hop_step<1>(w, a, st, acc);
    hop_step<2>(w, a, st, acc);
    hop_step<3>(w, a, st, acc);
    hop_step<4>(w, a, st, acc);
    hop_step<5>(w, a, st, acc);
    hop_step<6>(w, a, st, acc);
    hop_step<7>(w, a, st, acc);
    __builtin_amdgcn_sched_barrier(0);
    {   // clover, its diagonal, the largest term, last: fewest roundings at its size; the hopping
        // sum enters with -1/2
        const double2* C = (w.par ? a.C1 : a.C0) + w.cb;
        const uint32_t Vh = (uint32_t)g.Vh;
        double2 m[2][18];
#pragma unroll
        for (int e = 0; e < 18; ++e) m[0][e] = C[(uint32_t)e * Vh];
        place(w, st);
        const D2* v0 = w.buf + w.lane * PAD;
#pragma unroll
        for (int e = 0; e < 18; ++e) m[1][e] = C[(uint32_t)(18 + e) * Vh];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            D2 v[6];
#pragma unroll
            for (int e = 0; e < 6; ++e) {
                v[e] = v0[b * 6 + e];
                acc[b * 6 + e] *= -0.5;
            }
#pragma unroll
            for (int hi = 1; hi < 6; ++hi) {
#pragma unroll
                for (int lo = 0; lo < hi; ++lo) {
                    const double2 u = m[b][3 + hi * (hi - 1) / 2 + lo];
                    add_mul(acc[b * 6 + hi], u.x, u.y, v[lo]);
                    add_mul(acc[b * 6 + lo], u.x, -u.y, v[hi]);
                }
            }
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                add_re(acc[b * 6 + 2 * e], m[b][e].x, v[2 * e]);
                add_re(acc[b * 6 + 2 * e + 1], m[b][e].y, v[2 * e + 1]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // out through the same buffer
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int e = 0; e < 12; ++e) w.buf[w.lane * PAD + e] = acc[e];
    __builtin_amdgcn_wave_barrier();
    double2* o = a.out + rs + ((long)(w.t * g.Z + w.z) * w.plane + s0) * 12;
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        const int e = 64 * k + w.lane;
        if (e <= w.e1) *(D2*)&o[e] = w.buf[w.pos[k % 3] + k / 3 * 16 * PAD];
    }
}

}  // namespace

hipError_t launch_dirac(DiracArgs a, hipStream_t s) {
    if (a.nrhs <= 0) return hipSuccess;
    const Geo& g = a.g;
    const long plane = (long)g.Y * g.X, pw = (plane + 63) / 64;
    // A wave per 64 sites when these are mostly there (planes of 32 and more) and make a wave per
    // CU; four lanes per site below.  Four lanes, 64 sites (us per call): 8^3 x 16 with one
    // right-hand side 26, 30, with four 31.1, 30.9; 4x6x8 x 20 with five 29.8, 29.6; 6^3 x 24 with
    // four 29.0, 28.9, with 24 70, 57; 4^3 x 38 (16 sites per plane) with 100 101, 138; 24^3 x 48
    // with 12 3210, 1702.  The links' 32-bit byte offsets end at 7.2 million sites per parity.
    const bool sites = 2 * plane >= 64 * pw && 2L * g.Vh * a.nrhs >= 19200 && 37L * 16 * g.Vh < (1L << 32);
    const int per = std::min(a.nrhs, 12);
    a.ng = per;
    a.nT = g.T % 8 == 0 ? 8 : (g.T % 4 == 0 ? 4 : 2);
    const int ntm = g.T / a.nT, nZ = 8 / a.nT, nzm = (g.Z + nZ - 1) / nZ;
    // sites of a strip: an XCD's timeslices of three z planes for up to 12 right-hand sides in
    // 8 MB (of 2, 4, 8, 16 MB at 24^3 x 48 the best by 4%; 12 right-hand sides together 1.7 ms,
    // two 2.0, one 2.6: they share the links)
    const long l2 = (8L << 20) / (3L * ntm * per * 192);
    if (sites) {
        a.nstrip = (int)((pw + std::max(1L, l2 / 64) - 1) / std::max(1L, l2 / 64));
        a.nch = (int)((pw + a.nstrip - 1) / a.nstrip);
    } else {
        const int step = 16 / std::gcd(g.X, 16);  // rows that fill whole waves
        a.R = (int)std::min<long>(std::max<long>(step, l2 / g.X / step * step), g.Y);
        a.nstrip = (g.Y + a.R - 1) / a.R;
        a.nch = (a.R * g.X + 15) / 16;
    }
    // a launch's 32-bit grid ends at 2^32 threads, 512 per wave of an XCD
    const long group = (long)a.nstrip * nzm * ntm * a.nch * a.ng, most = std::max(1L, (1L << 23) / group - 1) * per;
    const int all = a.nrhs;
    for (long r0 = 0; r0 < all; r0 += most) {
        a.nrhs = (int)std::min(most, all - r0);
        const long waves = (a.nrhs + per - 1) / per * group;
        const dim3 grid((unsigned)((waves + 3) / 4 * 8));
        if (sites) hipLaunchKernelGGL(k_dirac_sites, grid, dim3(256), 0, s, a);
        else hipLaunchKernelGGL(k_dirac, grid, dim3(256), 0, s, a);
        a.in += a.nrhs * 24L * g.Vh;
        a.out += a.nrhs * 24L * g.Vh;
    }
    return hipGetLastError();
}

}  // namespace dlma
