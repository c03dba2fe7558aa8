// BiCGStab's vector steps, the FP64 conversions and the gauge copies on right-hand-side
// tiles (tile.h).
#include "tile_dev.h"

namespace dlma {

// ---------------------------------------------------------------- vector steps

// The steps of bicg.hip: lane (q, n) works on spin q of right-hand side n, a wave on one
// site of one tile, 768 contiguous bytes per field; the scalars of the lane's right-hand
// side stay in registers.  Streams bound by memory, in FP64 arithmetic; the x, r, p update
// of 8x20x20x18 with 60 right-hand sides, 708 MB, takes 114 us (128 us with loads and stores
// past the caches: fields of one solve often fit the 256 MB on the memory side).
template <int MODE>
__global__ void __launch_bounds__(256) k_tile_vec(const TileVecJob* __restrict__ jobs, int njob) {
    constexpr int NQ = MODE == BV_XRP ? 1 : 2;
    const int bid = blockIdx.x;
    int jb = 0;
    while (jb + 1 < njob && bid >= jobs[jb + 1].blk0) ++jb;
    const TileVecJob& J = jobs[jb];
    const int lb = bid - J.blk0, tile = lb / J.nsb, sb = lb - tile * J.nsb;
    const int lane = (int)threadIdx.x & 63, q = lane >> 4, n = lane & 15;
    const int wave = wave_uniform((int)threadIdx.x >> 6);
    const int r = tile * TILE + n, rc = r < J.nrhs ? r : 0;
    const bool use = r < J.nrhs && J.active[rc] != 0;
    double* part = MODE == BV_SH ? J.part_s : J.part;
    if (__ballot(use) == 0) {  // the whole block: zero partials
        if ((int)threadIdx.x < 16 * NQ) {
            const int c = (int)threadIdx.x & 15, k = (int)threadIdx.x >> 4;
            if (tile * TILE + c < J.nrhs) part[((size_t)(tile * TILE + c) * NQ + k) * J.pstride + sb] = 0.0;
        }
        return;
    }
    const int Vh = J.Vh;
    const uint32_t lane12 = 12u * (uint32_t)lane;
    auto load = [&](const WSrc& f, int cb, double v[6]) {
        const u32x3 w = wld3(f, lane12, 768u * (uint32_t)cb);
#pragma unroll
        for (int e = 0; e < 3; ++e) {
            const uint32_t x = w[e];
            v[2 * e] = word_lo(x);
            v[2 * e + 1] = word_hi(x);
        }
    };
    auto store = [&](const WSrc& f, int cb, bool on, const double v[6], uint32_t w[3]) {
#pragma unroll
        for (int e = 0; e < 3; ++e) w[e] = pack16((float)v[2 * e], (float)v[2 * e + 1]);
        if (on) {
            wide_store_begin();
            wst3<CP_DEFAULT>(f, lane12, 768u * (uint32_t)cb, (u32x3){w[0], w[1], w[2]});
            wide_store_end();
        }
    };
    const WSrc fr = tile_src(J.r, Vh, tile), fs = tile_src(J.s, Vh, tile), fv = tile_src(J.v, Vh, tile);
    const WSrc ft = tile_src(J.t, Vh, tile), fp = tile_src(J.p, Vh, tile), fx = tile_src(J.x, Vh, tile);
    const WSrc RH = wsrc(J.rh, 48u * (uint32_t)Vh);
    double al[2] = {0, 0}, om[2] = {0, 0}, be[2] = {0, 0};
    if (MODE != BV_RR) { al[0] = J.alpha[rc].x; al[1] = J.alpha[rc].y; }
    if (MODE == BV_XRP) {
        om[0] = J.omega[rc].x; om[1] = J.omega[rc].y;
        be[0] = J.beta[rc].x; be[1] = J.beta[rc].y;
    }
    const int reach = MODE == BV_SH ? 3 : 5;
    double q0 = 0, q1 = 0;
    const int c1 = min(Vh, (sb + 1) * J.sites);
    for (int cb = sb * J.sites + wave; cb < c1; cb += 4) {
        // first pass: beyond the reach of the outputs everything is zero and stays so
        const bool near = MODE == BV_RR || in_reach(J.tdist, J.titer, J.T, rc, J.tdist ? cb / J.vt : 0, reach);
        const bool on = use && near;
        if (__ballot(on) == 0) continue;
        double a[6], b[6], c[6];
        uint32_t w[3], rw[3];
        if (MODE == BV_RR || MODE == BV_SH) {
            const u32x3 h = wld3(RH, 12u * (uint32_t)q, 48u * (uint32_t)cb);
            rw[0] = h.x; rw[1] = h.y; rw[2] = h.z;
        }
        if (MODE == BV_RR) {  // (rh, r)
            const u32x3 h = wld3(fr, lane12, 768u * (uint32_t)cb);
            w[0] = h.x; w[1] = h.y; w[2] = h.z;
        } else if (MODE == BV_SH) {  // s = r - alpha v, and (rh, s) of the stored s
            load(fr, cb, a);
            load(fv, cb, b);
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                c[2 * e] = a[2 * e] - (al[0] * b[2 * e] - al[1] * b[2 * e + 1]);
                c[2 * e + 1] = a[2 * e + 1] - (al[0] * b[2 * e + 1] + al[1] * b[2 * e]);
            }
            store(fs, cb, on, c, w);
        }
        if (MODE == BV_RR || MODE == BV_SH) {
            double re = 0, im = 0;
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                const double ar = word_lo(rw[e]), ai = word_hi(rw[e]), sr = word_lo(w[e]), si = word_hi(w[e]);
                re += ar * sr + ai * si;
                im += ar * si - ai * sr;
            }
            if (on) {
                q0 += re;
                q1 += im;
            }
        }
        if (MODE == BV_XRP) {  // x += alpha p + omega s; r = s - omega t; p = r + beta (p - omega v); |r|^2
            double d[6], f[6];
            load(fx, cb, a);
            load(fp, cb, b);
            load(fs, cb, c);
            load(ft, cb, d);
            load(fv, cb, f);
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                const int i = 2 * e, j = 2 * e + 1;
                a[i] += al[0] * b[i] - al[1] * b[j] + om[0] * c[i] - om[1] * c[j];
                a[j] += al[0] * b[j] + al[1] * b[i] + om[0] * c[j] + om[1] * c[i];
                c[i] -= om[0] * d[i] - om[1] * d[j];
                c[j] -= om[0] * d[j] + om[1] * d[i];
                const double gr = b[i] - (om[0] * f[i] - om[1] * f[j]), gi = b[j] - (om[0] * f[j] + om[1] * f[i]);
                b[i] = c[i] + be[0] * gr - be[1] * gi;
                b[j] = c[j] + be[0] * gi + be[1] * gr;
            }
            store(fx, cb, on, a, w);
            store(fr, cb, on, c, w);
            store(fp, cb, on, b, w);
            double s2 = 0;
#pragma unroll
            for (int e = 0; e < 6; ++e) s2 += c[e] * c[e];
            if (on) q0 += s2;
        }
    }
    __shared__ double sm[4][2][16];
    q0 = sum_over_q(q0);
    if (NQ > 1) q1 = sum_over_q(q1);
    if (q == 0) {
        sm[wave][0][n] = q0;
        sm[wave][1][n] = q1;
    }
    __syncthreads();
    if ((int)threadIdx.x < 16 * NQ) {
        const int c = (int)threadIdx.x & 15, k = (int)threadIdx.x >> 4;
        if (tile * TILE + c < J.nrhs)
            part[((size_t)(tile * TILE + c) * NQ + k) * J.pstride + sb] = ((sm[0][k][c] + sm[1][k][c]) + sm[2][k][c]) + sm[3][k][c];
    }
}

hipError_t launch_tile_vec(const TileVecJob* d, int njob, int nblocks, int mode, hipStream_t s) {
    if (nblocks <= 0) return hipSuccess;
    switch (mode) {
    case BV_RR: hipLaunchKernelGGL((k_tile_vec<BV_RR>), dim3(nblocks), dim3(256), 0, s, d, njob); break;
    case BV_SH: hipLaunchKernelGGL((k_tile_vec<BV_SH>), dim3(nblocks), dim3(256), 0, s, d, njob); break;
    case BV_XRP: hipLaunchKernelGGL((k_tile_vec<BV_XRP>), dim3(nblocks), dim3(256), 0, s, d, njob); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------- conversions

// A block takes 32 sites of one tile, a thread one (right-hand side, site): the FP64 planes
// are read in runs of 32 sites, and the words pass through LDS so that a tile's sites are
// written as one contiguous span.
__global__ void __launch_bounds__(TILE * TCONV_SITES) k_tile_conv(const TileConvJob* __restrict__ jobs, int njob) {
    const int bid = blockIdx.x;
    int jb = 0;
    while (jb + 1 < njob && bid >= jobs[jb + 1].blk0) ++jb;
    const TileConvJob& J = jobs[jb];
    const int lb = bid - J.blk0, tile = lb / J.nsb, sb = lb - tile * J.nsb;
    const int n = (int)threadIdx.x / TCONV_SITES, i = (int)threadIdx.x % TCONV_SITES;
    const int r = tile * TILE + n, cb0 = sb * TCONV_SITES, cb = cb0 + i;
    const bool use = r < J.nrhs && J.active[r] != 0;
    __shared__ uint32_t words[TCONV_SITES * 192];
    __shared__ int act[TILE];
    double nrm = 0.0;
    uint32_t w[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) w[c] = 0;
    if (use && cb < J.Vh && tsup_any(J.tsup, J.T, r, J.vt > 0 ? cb / J.vt : 0, J.tdil)) {
        double x[24];
        load_spinor<P64, double>(J.src, J.Vh, r, cb, x);
        const double n2 = J.s[r], f = n2 > 0 ? 1.0 / sqrt(n2) : 0.0;
        float y[24];
#pragma unroll
        for (int k = 0; k < 24; ++k) {
            y[k] = (float)(x[k] * f);
            nrm += (double)y[k] * (double)y[k];
        }
#pragma unroll
        for (int c = 0; c < 12; ++c) w[c] = pack16(y[2 * c], y[2 * c + 1]);
    }
    // words[site][spin][rhs][colour]
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int c = 0; c < 3; ++c) words[i * 192 + (s * 16 + n) * 3 + c] = w[3 * s + c];
    if (i == 0) act[n] = use ? 1 : 0;
#pragma unroll
    for (int off = TCONV_SITES / 2; off > 0; off >>= 1) nrm += __shfl_xor(nrm, off, 64);
    if (i == 0 && r < J.nrhs) J.part[(size_t)r * J.pstride + sb] = nrm;
    __syncthreads();
    const int ns = min(TCONV_SITES, J.Vh - cb0);
    const size_t o = ((size_t)tile * J.Vh + cb0) * 192;
    for (int e = threadIdx.x; e < ns * 192; e += TILE * TCONV_SITES)
        if (act[e / 3 % 16]) {  // the others keep their fields (x is still needed)
            J.a[o + e] = words[e];
            J.b[o + e] = words[e];
            J.c[o + e] = 0;
        }
}

hipError_t launch_tile_conv(const TileConvJob* d, int njob, int nblocks, hipStream_t s) {
    if (nblocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_tile_conv, dim3(nblocks), dim3(TILE * TCONV_SITES), 0, s, d, njob);
    return hipGetLastError();
}

// a tile field to the layout of the FP64 kernels that read it (planes of bfloat16 words)
__global__ void __launch_bounds__(TILE * TCONV_SITES) k_tile_back(const TileBackJob* __restrict__ jobs, int njob) {
    const int bid = blockIdx.x;
    int jb = 0;
    while (jb + 1 < njob && bid >= jobs[jb + 1].blk0) ++jb;
    const TileBackJob& J = jobs[jb];
    const int lb = bid - J.blk0, tile = lb / J.nsb, sb = lb - tile * J.nsb;
    const int n = (int)threadIdx.x / TCONV_SITES, i = (int)threadIdx.x % TCONV_SITES;
    const int r = tile * TILE + n, cb0 = sb * TCONV_SITES, cb = cb0 + i, Vh = J.Vh;
    __shared__ uint32_t words[TCONV_SITES * 192];
    const int ns = min(TCONV_SITES, Vh - cb0);
    const size_t o = ((size_t)tile * Vh + cb0) * 192;
    for (int e = threadIdx.x; e < ns * 192; e += TILE * TCONV_SITES) words[e] = J.a[o + e];
    __syncthreads();
    if (r >= J.nrhs || cb >= Vh) return;
    uint32_t w[12];
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int c = 0; c < 3; ++c) w[3 * s + c] = words[i * 192 + (s * 16 + n) * 3 + c];
    uint32_t* v = J.v + (size_t)r * 12 * Vh;
#pragma unroll
    for (int c = 0; c < 12; ++c) v[(size_t)c * Vh + cb] = w[c];
}

hipError_t launch_tile_back(const TileBackJob* d, int njob, int nblocks, hipStream_t s) {
    if (nblocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_tile_back, dim3(nblocks), dim3(TILE * TCONV_SITES), 0, s, d, njob);
    return hipGetLastError();
}

// ---------------------------------------------------------------- gauge copies

// word (site, direction, row, col) of the matrices acting on the neighbours
__global__ void k_tile_links(const double2* __restrict__ U64, Geo g, int par, uint32_t* __restrict__ L) {
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i >= 72L * g.Vh) return;
    const int site = (int)(i / 72), e = (int)(i - 72L * site), d = e / 9, a = e % 9 / 3, b = e % 3;
    const int mu = d >> 1;
    double2 u;
    if ((d & 1) == 0) {
        u = U64[((size_t)(par * 4 + mu) * 9 + a * 3 + b) * g.Vh + site];
    } else {
        const Nbr nb = neighbours(g, par, site);
        u = U64[((size_t)((1 - par) * 4 + mu) * 9 + b * 3 + a) * g.Vh + nb.n[d]];
        u.y = -u.y;
    }
    L[144L * site + e] = pack16((float)u.x, (float)u.y);
}
hipError_t launch_tile_links(const double2* U64, const Geo& g, int par, uint32_t* L, hipStream_t s) {
    hipLaunchKernelGGL(k_tile_links, dim3((unsigned)((72L * g.Vh + 255) / 256)), dim3(256), 0, s, U64, g, par, L);
    return hipGetLastError();
}

// both triangles of the packed Hermitian blocks
__global__ void k_tile_clover(const double2* __restrict__ C64, int Vh, uint32_t* __restrict__ L) {
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i >= 72L * Vh) return;
    const int site = (int)(i / 72), e = (int)(i - 72L * site), blk = e / 36, a = e % 36 / 6, b = e % 6;
    const double2* src = C64 + (size_t)blk * 18 * Vh + site;
    double2 v;
    if (a == b) {
        const double2 d = src[(size_t)(a >> 1) * Vh];
        v = make_double2((a & 1) ? d.y : d.x, 0.0);
    } else {
        const int hi = a > b ? a : b, lo = a > b ? b : a;
        v = src[(size_t)(3 + hi * (hi - 1) / 2 + lo) * Vh];
        if (a < b) v.y = -v.y;
    }
    L[144L * site + 72 + e] = pack16((float)v.x, (float)v.y);
}
hipError_t launch_tile_clover(const double2* C64, int Vh, uint32_t* L, hipStream_t s) {
    hipLaunchKernelGGL(k_tile_clover, dim3((unsigned)((72L * Vh + 255) / 256)), dim3(256), 0, s, C64, Vh, L);
    return hipGetLastError();
}

// the numbers of k_fill_random for one field, as the shared shadow residual
__global__ void k_tile_random(uint32_t* __restrict__ f, int Vh, unsigned seed) {
    const int cb = (int)(blockIdx.x * 256 + threadIdx.x);
    if (cb >= Vh) return;
    float v[24];
    for (int k = 0; k < 24; ++k) {
        uint64_t z = (uint64_t)seed * 0x9E3779B97F4A7C15ull + (uint64_t)((long)cb * 24 + k) + 1;
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        z ^= z >> 31;
        v[k] = (float)((double)(z >> 11) * (1.0 / 9007199254740992.0) - 0.5);
    }
    for (int c = 0; c < 12; ++c) f[(size_t)cb * 12 + c] = pack16(v[2 * c], v[2 * c + 1]);
}
hipError_t launch_tile_random(uint32_t* f, int Vh, unsigned seed, hipStream_t s) {
    hipLaunchKernelGGL(k_tile_random, dim3((unsigned)((Vh + 255) / 256)), dim3(256), 0, s, f, Vh, seed);
    return hipGetLastError();
}

}  // namespace dlma
