// Timeslice contractions behind the correlators (paper eq. 2-4).  With the four
// spin-diluted solutions of a source group as columns i = (label s', spin a) of 3 L^3
// rows (site, colour) on a timeslice, everything the correlators need is
//   tau[k][i]  = sum_rows conj(v_k) F_i            (projections on the Laplacian modes;
//                                                   for distillation the perambulator)
//   gram[i][j] = sum_groups sum_rows conj(A_i) B_j  (spin-resolved inner products)
//   proj[i][j] = sum_groups sum_k conj(tauA[k][i]) tauB[k][j]
// for (A, B) = (dist, dist), (phi, phi), (phibar, phi); the pieces are fixed linear
// combinations of the 16 x 16 sums, formed by k_corr_pieces.
// Spinor fields are canonical complex128 [T][Z][Y][X][4][3]; V is [T][nev][L^3][3].
#include "laplace.h"

namespace dlma {

// ---------------------------------------------------------------- projections and Grams
//
// One wave takes two column sets (two distillation groups, or the phi and phibar of a
// noise group) on one chunk of sites of a timeslice, and up to 32 modes, on FP64 matrix
// instructions (v_mfma_f64_16x16x4: operand lane l holds row or column l % 16 at
// k = l / 16, result register i of lane l is row 4 i + l / 16 of column l % 16).  Lane
// (q, m) = (l / 16, l % 16) loads the three colours of site x + q of column m (or of
// mode m): 48 contiguous bytes, four sites of four spins contiguous across the wave.
// The same registers are the A and the B operand of the Gram, so nothing is shuffled and
// every field is read once for both results.  Two column sets per wave halve the reads
// of V (L2 hits: the waves of a block take consecutive groups of one chunk, and each
// XCD walks a contiguous range of chunks).
// A step's twelve products are summed among themselves and then added: a rounding at the
// size of the sum for every twelve terms.  The next step's numbers are loaded while one is
// worked on.
// Bound: the matrix cores (64 cycles per instruction, 8 flop per complex product; two waves
// per SIMD at 220 registers with the Grams and 32 modes).  At
// 16^3 x 32 with 32 modes, 128 distillation and 32 noise solutions the projections and
// Grams took 23.8 ms as one block per field and four modes, every field read nev / 4
// times for tau and 8 times for the Grams, and the sums over groups and spins 43 ms on
// the host (67.2 ms per call); now 1.64 ms per call, 89 GFLOP in matrix instructions: 54
// TFLOP/s over the call, of a 64 TFLOP/s FP64 matrix product.  Without the next step's loads
// under way 1.72 ms; 24x12^3 with 48 modes 1.26, 1.17.
typedef double d4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double2 cconjmul(double2 a, double2 b) { return make_double2(a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x); }
__device__ __forceinline__ d4 mma64(double a, double b, d4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

// sums over four sites and three colours of conj(a) b: real or imaginary parts
__device__ __forceinline__ d4 dot12(const double2 (&a)[3], const double2 (&b)[3], bool im) {
    d4 r = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        r = mma64(a[c].x, im ? b[c].y : b[c].x, r);
        r = mma64(im ? -a[c].y : a[c].y, im ? b[c].x : b[c].y, r);
    }
    return r;
}
// and of Re(a) Im(a)
__device__ __forceinline__ d4 cross12(const double2 (&a)[3]) {
    d4 r = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int c = 0; c < 3; ++c) r = mma64(a[c].x, a[c].y, r);
    return r;
}

// Result tile (re, im) of one wave into [16][16] complex numbers, rows limited to nrow
__device__ __forceinline__ void store_tile(double2* o, int lane, int nrow, const d4& re, const d4& im) {
    const int q = lane >> 4, m = lane & 15;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (4 * i + q < nrow) o[(4 * i + q) * 16 + m] = make_double2(re[i], im[i]);
}

template <bool NOISE, bool GRAM, int MT>
__global__ void __launch_bounds__(256, GRAM ? 2 : 1) k_contract(ContractArgs a) {
    // block -> (unit group fastest, site chunk, timeslice), contiguous per XCD
    const int per = gridDim.x >> 3;
    const int lb = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    const int nub = (a.nunit + 3) / 4;
    const int ub = lb % nub, r = lb / nub;
    const int rk = r / a.nkb, kc = rk % a.ks, ti = rk / a.ks;
    const int k0 = a.k0 + (r - rk * a.nkb) * 16 * MT;  // first of this wave's modes
    const int unit = ub * 4 + (int)(threadIdx.x >> 6);
    if (ti >= a.nt || unit >= a.nunit) return;  // whole waves
    const int t = a.tlist ? a.tlist[ti] : a.t0 + ti;
    const int lane = (int)threadIdx.x & 63, q = lane >> 4, m = lane & 15;
    const long L3 = a.L3;
    const long x0 = kc * a.chunk, x1 = x0 + a.chunk < L3 ? x0 + a.chunk : L3;
    // column sets: groups 2 unit, 2 unit + 1 (the second repeats the first past the end), or phi and phibar
    const int g0 = NOISE ? unit : 2 * unit;
    const bool two = NOISE || g0 + 1 < a.ng;
    const long col = ((long)t * L3 + x0 + q) * 12 + (m & 3) * 3;
    auto field = [&](int g) { return (long)min(g * 4 + (m >> 2), a.nf - 1) * a.fs + col; };
    const double2* p0 = a.f0 + field(g0);
    const double2* p1 = NOISE ? a.f1 + field(g0) : a.f0 + field(two ? g0 + 1 : g0);
    const double2* pv[MT];
#pragma unroll
    for (int b = 0; b < MT; ++b) {
        const int k = k0 + 16 * b + m;  // modes past the last repeat it; their rows are not stored
        pv[b] = a.Vall + (((long)(t - a.tv0) * a.nev + (k < a.nev ? k : a.nev - 1)) * L3 + x0 + q) * 3;
    }
    const d4 z = {0.0, 0.0, 0.0, 0.0};
    d4 tr[2][MT], tm[2][MT], g00r = z, g00x = z, g10r = z, g10i = z;
#pragma unroll
    for (int b = 0; b < MT; ++b) { tr[0][b] = z; tr[1][b] = z; tm[0][b] = z; tm[1][b] = z; }
    double2 f0[3], f1[3], v[MT][3];
    auto load = [&] {
#pragma unroll
        for (int c = 0; c < 3; ++c) { f0[c] = p0[c]; f1[c] = p1[c]; }
#pragma unroll
        for (int b = 0; b < MT; ++b)
#pragma unroll
            for (int c = 0; c < 3; ++c) v[b][c] = pv[b][c];
        p0 += 48;
        p1 += 48;
#pragma unroll
        for (int b = 0; b < MT; ++b) pv[b] += 12;
    };
    if (x0 < x1) load();
    for (long x = x0; x < x1; x += 4) {
        double2 c0[3], c1[3], cv[MT][3];
#pragma unroll
        for (int c = 0; c < 3; ++c) { c0[c] = f0[c]; c1[c] = f1[c]; }
#pragma unroll
        for (int b = 0; b < MT; ++b)
#pragma unroll
            for (int c = 0; c < 3; ++c) cv[b][c] = v[b][c];
        if (x + 4 < x1) load();  // the next step's, while this one is worked on
        // twelve products at a time are summed among themselves before they join the sum: a
        // rounding at its size for every twelve terms
#pragma unroll
        for (int b = 0; b < MT; ++b) {
            tr[0][b] += dot12(cv[b], c0, false);
            tm[0][b] += dot12(cv[b], c0, true);
            tr[1][b] += dot12(cv[b], c1, false);
            tm[1][b] += dot12(cv[b], c1, true);
        }
        if (GRAM) {
            // (A, A): the imaginary part is X - X^T with X = Re(A)^T Im(A)
            g00r += dot12(c0, c0, false);
            g00x += cross12(c0);
            if (NOISE) {
                g10r += dot12(c1, c0, false);
                g10i += dot12(c1, c0, true);
            } else if (two) {
                g00r += dot12(c1, c1, false);
                g00x += cross12(c1);
            }
        }
    }
    const int nset = NOISE ? 2 * a.ng : a.ng;
#pragma unroll
    for (int s = 0; s < 2; ++s)
        if (s == 0 || two)
#pragma unroll
            for (int b = 0; b < MT; ++b) {
                const int k = k0 + 16 * b;
                const int set = NOISE ? 2 * g0 + s : g0 + s;
                if (k < a.nev)
                    store_tile(a.taup + ((((long)kc * nset + set) * a.nt + ti) * a.nev + k) * 16, lane, a.nev - k, tr[s][b], tm[s][b]);
            }
    if (GRAM) {
        constexpr int NG = NOISE ? 2 : 1;
        double2* o = a.gramp + (((long)ti * a.ks + kc) * a.nunit + unit) * NG * 256;
        store_tile(o, lane, 16, g00r, g00x);
        if (NOISE) store_tile(o + 256, lane, 16, g10r, g10i);
    }
}

// Site chunks per (unit, timeslice): about 4096 waves in all (eight per SIMD slot pair),
// at least 16 steps of four sites each, or 4 while there are fewer than 64 chunks
static int contract_chunks(long L3, long waves) {
    const long want = (4096 + waves - 1) / waves, most = std::max(1L, std::max(L3 / 64, std::min(L3 / 16, 64L)));
    return (int)(want < 1 ? 1 : (want > most ? most : want));
}

int contract_ks(const Geo& g, int nt, int units) {
    return contract_chunks((long)g.Z * g.Y * g.X, (long)std::max(1, nt) * std::max(1, units));
}

template <bool NOISE> static hipError_t launch_contract_t(ContractArgs a, bool gram, hipStream_t s) {
    if (a.nev <= 0) return hipSuccess;
    const dim3 block(256);
    auto grid = [&] { return dim3((unsigned)(((long)a.nt * a.ks * ((a.nunit + 3) / 4) * a.nkb + 7) / 8 * 8)); };
    a.k0 = 0;
    a.nkb = 1;
    if (gram) {  // with the first modes
        if (a.nev <= 16) hipLaunchKernelGGL((k_contract<NOISE, true, 1>), grid(), block, 0, s, a);
        else hipLaunchKernelGGL((k_contract<NOISE, true, 2>), grid(), block, 0, s, a);
        a.k0 = 32;
    }
    const int left = a.nev - a.k0;
    if (left <= 0) return hipGetLastError();
    // 32 modes per wave halve the reads of the fields; 16 while there are too few waves
    const bool one = left <= 16 || (long)a.nt * a.ks * a.nunit * ((left + 31) / 32) < 1024;
    a.nkb = one ? (left + 15) / 16 : (left + 31) / 32;
    if (one) hipLaunchKernelGGL((k_contract<NOISE, false, 1>), grid(), block, 0, s, a);
    else hipLaunchKernelGGL((k_contract<NOISE, false, 2>), grid(), block, 0, s, a);
    return hipGetLastError();
}

// tau[i] = sum of its ks partials: 16 values per block at a time, sixteen slices of the partials each
__global__ void __launch_bounds__(256) k_sum_parts(const double2* __restrict__ p, long n, int ks, double2* __restrict__ o) {
    __shared__ double2 sm[16][16];
    const int e = (int)threadIdx.x & 15, sl = (int)threadIdx.x >> 4;
    for (long i = (long)blockIdx.x * 16 + e; i < n; i += (long)gridDim.x * 16) {  // n is a multiple of 16
        double2 v = make_double2(0.0, 0.0);
#pragma unroll 4
        for (int k = sl; k < ks; k += 16) {
            const double2 w = p[i + k * n];
            v.x += w.x;
            v.y += w.y;
        }
        sm[sl][e] = v;
        __syncthreads();
        for (int half = 8; half > 0; half >>= 1) {  // pairwise
            if (sl < half) {
                v.x += sm[sl + half][e].x;
                v.y += sm[sl + half][e].y;
                sm[sl][e] = v;
            }
            __syncthreads();
        }
        if (sl == 0) o[i] = v;
    }
}

hipError_t launch_contract(const ContractArgs& a0, bool noise, bool gram, double2* tau, hipStream_t s) {
    if (a0.ng <= 0 || a0.nt <= 0) return hipSuccess;
    ContractArgs a = a0;
    a.nunit = noise ? a.ng : (a.ng + 1) / 2;
    a.chunk = ((a.L3 + a.ks - 1) / a.ks + 3) / 4 * 4;  // L3 is a multiple of 8
    if (a.ks == 1) a.taup = tau;
    const hipError_t e = noise ? launch_contract_t<true>(a, gram, s) : launch_contract_t<false>(a, gram, s);
    if (e != hipSuccess || a.ks == 1) return e;
    const long n = (long)(noise ? 2 : 1) * a.ng * a.nt * a.nev * 16;
    // (a launch ends at 2^32 threads)
    hipLaunchKernelGGL(k_sum_parts, dim3((unsigned)std::min(n / 16, 1L << 20)), dim3(256), 0, s, a.taup, n, a.ks, tau);
    return hipGetLastError();
}

// proj[i][j] partials: wave w of block (., timeslice) adds groups w, w + nw, ... of
// conj(tauA[k][i]) tauB[k][j] over the modes, four modes per matrix instruction (rows
// past the last mode enter as zero).  A and B are sets oa + st g, ob + st g of tau.
__global__ void __launch_bounds__(256) k_proj_gram(const double2* __restrict__ tau, int nt, int nev, int ng, int oa, int ob, int st,
                                                   double2* __restrict__ part) {
    const int ti = blockIdx.y, nw = gridDim.x * 4, w = blockIdx.x * 4 + (int)(threadIdx.x >> 6);
    const int lane = (int)threadIdx.x & 63, q = lane >> 4, m = lane & 15;
    d4 re = {0.0, 0.0, 0.0, 0.0}, im = re;
    for (int g = w; g < ng; g += nw) {
        const double2* A = tau + ((long)(oa + st * g) * nt + ti) * nev * 16 + m;
        const double2* B = tau + ((long)(ob + st * g) * nt + ti) * nev * 16 + m;
        for (int k0 = 0; k0 < nev; k0 += 4) {
            const bool ok = k0 + q < nev;
            const double2 x = ok ? A[(long)(k0 + q) * 16] : make_double2(0.0, 0.0);
            const double2 y = ok ? B[(long)(k0 + q) * 16] : make_double2(0.0, 0.0);
            re = mma64(x.x, y.x, re);
            im = mma64(x.x, y.y, im);
            re = mma64(x.y, y.y, re);
            im = mma64(-x.y, y.x, im);
        }
    }
    store_tile(part + ((long)ti * nw + w) * 256, lane, 16, re, im);
}

constexpr int PROJ_BLOCKS = 4;  // k_proj_gram blocks per timeslice (16 partials)

// C[gamma][part][delta] from the partial sums of the three Grams and their projected
// forms, block delta: thread e = (i, j) of four slices adds its entry over the partials,
// W[gamma][e] holds the piece's spin weights sum_Gamma N[s][s'] M[a][b] / (Gammas).  A chain
// of sums: a wave per (gamma, part) with shuffles, 20 us; the whole block on each in turn, two
// barriers apiece, took 80 us.
__global__ void __launch_bounds__(1024) k_corr_pieces(CorrPiecesArgs a) {
    __shared__ double2 sm[4][256];
    __shared__ double2 pc[DLMA_NPARTS][256];
    const int d = blockIdx.x, T = a.T, t = (a.t_src + d) % T;
    const int e = (int)threadIdx.x & 255, sl = (int)threadIdx.x >> 8;
    const int eT = (e & 15) * 16 + (e >> 4);
    // F: 0 dist, 1 (phi, phi), 2 (phibar, phi); [0] whole, [1] projected
    double2 F[3][2];
    auto sum = [&](const double2* p, int n, long stride, int ent) {
        __syncthreads();  // the previous sum has been read
        double2 v = make_double2(0.0, 0.0);
        for (int k = sl; k < n; k += 4) {
            const double2 w = p[k * stride + ent];
            v.x += w.x;
            v.y += w.y;
        }
        sm[sl][ent] = v;
        __syncthreads();
        double2 s = sm[0][ent];
        for (int k = 1; k < 4; ++k) {
            s.x += sm[k][ent].x;
            s.y += sm[k][ent].y;
        }
        return s;
    };
    auto hermitian = [&](double2 v) {  // (re, X) -> (re, X - X^T)
        __syncthreads();
        if (sl == 0) sm[0][e] = v;
        __syncthreads();
        return make_double2(v.x, v.y - sm[0][eT].y);
    };
    const double2 z = make_double2(0.0, 0.0);
    for (int k = 0; k < 3; ++k) F[k][0] = F[k][1] = z;
    const int np = PROJ_BLOCKS * 4;
    if (a.nud > 0) {
        F[0][0] = hermitian(sum(a.gd + (long)t * a.nud * 256, a.nud, 256, e));
        F[0][1] = sum(a.pd + (long)t * np * 256, np, 256, e);
    }
    if (a.nun > 0) {
        F[1][0] = hermitian(sum(a.gn + (long)t * a.nun * 512, a.nun, 512, e));
        F[2][0] = sum(a.gn + (long)t * a.nun * 512 + 256, a.nun, 512, e);
        F[1][1] = sum(a.pn + (long)t * np * 256, np, 256, e);
        F[2][1] = sum(a.pq + (long)t * np * 256, np, 256, e);
    }
    auto sub = [](double2 x, double2 y) { return make_double2(x.x - y.x, x.y - y.y); };
    const double2 piece[DLMA_NPARTS] = {sub(F[2][0], F[2][1]), F[2][1], sub(sub(F[1][0], F[2][0]), sub(F[1][1], F[2][1])),
                                        sub(F[1][1], F[2][1]), F[1][0], F[0][1], sub(F[0][0], F[0][1])};
    if (sl == 0)
        for (int p = 0; p < DLMA_NPARTS; ++p) pc[p][e] = piece[p];
    __syncthreads();
    // one wave per (gamma, part)
    const int lane = (int)threadIdx.x & 63;
    for (int o = (int)threadIdx.x >> 6; o < DLMA_NGAMMA * DLMA_NPARTS; o += 16) {
        const int gi = o / DLMA_NPARTS, p = o - gi * DLMA_NPARTS;
        double re = 0.0, im = 0.0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double2 w = a.W[gi * 256 + 64 * k + lane], c = pc[p][64 * k + lane];
            if (w.x != 0.0 || w.y != 0.0) {  // absent entries enter nothing, not even a NaN
                re += w.x * c.x - w.y * c.y;
                im += w.x * c.y + w.y * c.x;
            }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            re += __shfl_xor(re, off, 64);
            im += __shfl_xor(im, off, 64);
        }
        if (lane == 0) {
            const double s = p < 5 ? a.inv_nvec : 1.0;
            a.C[((long)gi * DLMA_NPARTS + p) * T + d] = make_double2(re * s, im * s);
        }
    }
}

int proj_gram_parts() { return PROJ_BLOCKS * 4; }

hipError_t launch_proj_gram(const double2* tau, int nt, int nev, int ng, int oa, int ob, int st, double2* part, hipStream_t s) {
    hipLaunchKernelGGL(k_proj_gram, dim3(PROJ_BLOCKS, nt), dim3(256), 0, s, tau, nt, nev, ng, oa, ob, st, part);
    return hipGetLastError();
}

hipError_t launch_corr_pieces(const CorrPiecesArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(k_corr_pieces, dim3(a.T), dim3(1024), 0, s, a);
    return hipGetLastError();
}

// re + i im += x w over four columns, summed among themselves first: a rounding at the size of
// the sum for every four terms
__device__ __forceinline__ void mac4(d4& re, d4& im, double2 x, double2 w) {
    const d4 z = {0.0, 0.0, 0.0, 0.0};
    re += mma64(-x.y, w.y, mma64(x.x, w.x, z));
    im += mma64(x.y, w.x, mma64(x.x, w.y, z));
}

// ---------------------------------------------------------------- projector
//
// box(t) in = sum_k v_k c_k with c = V^dag in on the contraction kernel (a right-hand side
// is a field, four of them a column set), then out = c V or in - c V on timeslice t as a
// matrix product (32 rows (site, colour) and four or eight right-hand sides per wave) in one
// launch with the zero fill of the other timeslices.  Bound: the fill, a stream of
// stores.  With a thread per (site, spin) storing 48 bytes apart and a block per (mode,
// right-hand side) for c, 32 modes and right-hand sides at 24^3 x 48 took 1.32 ms; 0.77 ms so
// (4.1 GB of stores: 5.3 TB/s over the call).
constexpr int FILL_PER_BLOCK = 1024;

template <int H>  // column sets per wave
__global__ void __launch_bounds__(256, H == 2 ? 1 : 4) k_proj_apply(const double2* __restrict__ Vt, const double2* in, double2* out, long L3, long fs,
                                                    int t, int nev, const double2* __restrict__ coef, int nrhs, int mode,
                                                    unsigned nab, unsigned nrb) {
    const long tofs = (long)t * L3 * 12;
    if (blockIdx.x >= nab) {  // zeros off the timeslice
        const unsigned fb = blockIdx.x - nab, nfb = (gridDim.x - nab) / (unsigned)nrhs;
        const unsigned r = fb / nfb;
        const long e0 = (long)(fb - r * nfb) * FILL_PER_BLOCK + threadIdx.x;
        double2* o = out + (long)r * fs;
#pragma unroll
        for (int k = 0; k < FILL_PER_BLOCK / 256; ++k) {
            const long e = e0 + k * 256;
            if (e < fs && (e < tofs || e >= tofs + L3 * 12)) o[e] = make_double2(0.0, 0.0);
        }
        return;
    }
    const int lane = (int)threadIdx.x & 63, q = lane >> 4, m = lane & 15;
    const long nrow = L3 * 3;
    const unsigned ub = blockIdx.x / nrb;  // right-hand sides 4 H ub ..
    const long r0 = ((long)(blockIdx.x - ub * nrb) * 4 + (threadIdx.x >> 6)) * 32;
    if (r0 >= nrow) return;  // whole waves
    long row[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const long r = r0 + 16 * b + m;
        row[b] = r < nrow ? r : nrow - 1;
    }
    const bool two = H == 2 && 8 * (int)ub + 4 < nrhs;
    const d4 z = {0.0, 0.0, 0.0, 0.0};
    d4 re[H][2], im[H][2];
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
        for (int b = 0; b < 2; ++b) re[h][b] = im[h][b] = z;
    const double2* v = Vt + (long)q * nrow;
    const double2* c = coef + ((long)ub * H * nev + q) * 16 + m;
    auto load = [&](int k, double2 (&x)[2], double2 (&w)[H]) {
#pragma unroll
        for (int b = 0; b < 2; ++b) x[b] = make_double2(0.0, 0.0);
#pragma unroll
        for (int h = 0; h < H; ++h) w[h] = make_double2(0.0, 0.0);
        if (k + q < nev) {
#pragma unroll
            for (int b = 0; b < 2; ++b) x[b] = v[(long)k * nrow + row[b]];
            w[0] = c[(long)k * 16];
            if (two) w[H - 1] = c[((long)nev + k) * 16];
        }
    };
    double2 x[2], w[H];
    if (H == 2) load(0, x, w);
    for (int k = 0; k < nev; k += 4) {
        // two column sets: the next four modes are on their way while these are worked on (24^3 x
        // 48 with 32 modes and right-hand sides 766 us per call, 778 without; one set would lose 3%)
        double2 nx[2], nw[H];
        if (H == 2) load(k + 4, nx, nw);
        else load(k, x, w);
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int b = 0; b < 2; ++b) mac4(re[h][b], im[h][b], x[b], w[h]);
        if (H == 2) {
#pragma unroll
            for (int b = 0; b < 2; ++b) x[b] = nx[b];
#pragma unroll
            for (int h = 0; h < H; ++h) w[h] = nw[h];
        }
    }
#pragma unroll
    for (int h = 0; h < H; ++h) {
        const int r = 4 * (H * (int)ub + h) + (m >> 2);
        if (r >= nrhs) continue;
        const long base = (long)r * fs + tofs + (m & 3) * 3;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const long rw = r0 + 16 * b + 4 * i + q;
                if (rw >= nrow) continue;
                const long e = base + rw / 3 * 12 + rw % 3;
                double2 o = make_double2(re[h][b][i], im[h][b][i]);
                if (mode == 1) {
                    const double2 x = in[e];
                    o = make_double2(x.x - o.x, x.y - o.y);
                }
                out[e] = o;
            }
    }
}

// c of one mode and one right-hand side per block, for few of them
__global__ void __launch_bounds__(256) k_proj_coef(const double2* __restrict__ Vt, const double2* __restrict__ in, long L3, long tofs,
                                                   long fs, int nev, double2* __restrict__ coef) {
    const int k = blockIdx.x, r = blockIdx.y;
    const double2* v = Vt + (long)k * L3 * 3;
    const double2* f = in + (long)r * fs + tofs;
    // thread (site, spin): 48 contiguous bytes, four sites' spins contiguous
    const int sp = (int)threadIdx.x & 3;
    double2 a = make_double2(0.0, 0.0);
#pragma unroll 4
    for (long x = threadIdx.x >> 2; x < L3; x += 64)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double2 p = cconjmul(v[x * 3 + c], f[(x * 4 + sp) * 3 + c]);
            a.x += p.x;
            a.y += p.y;
        }
    // over the sixteen sites of a wave, then the waves
#pragma unroll
    for (int off = 4; off < 64; off <<= 1) {
        a.x += __shfl_xor(a.x, off, 64);
        a.y += __shfl_xor(a.y, off, 64);
    }
    __shared__ double2 sm[4][4];
    const int lane = (int)threadIdx.x & 63;
    if (lane < 4) sm[threadIdx.x >> 6][lane] = a;
    __syncthreads();
    if (threadIdx.x < 4) {
        double2 t = sm[0][threadIdx.x];
        for (int w = 1; w < 4; ++w) {
            t.x += sm[w][threadIdx.x].x;
            t.y += sm[w][threadIdx.x].y;
        }
        coef[((long)(r >> 2) * nev + k) * 16 + (r & 3) * 4 + threadIdx.x] = t;
    }
}

// site chunks of c: 16 sites each (four steps of the contraction kernel, 1.5 us apiece), at
// most 256, and few enough that four right-hand sides' partials fit PROJ_PART_CAP
int project_ks(const Geo& g, int nev) {
    const long L3 = (long)g.Z * g.Y * g.X;
    const long k = std::min(std::min(L3 / 16, 256L), PROJ_PART_CAP / (16L * std::max(1, nev)));
    return (int)std::max(1L, k);
}

hipError_t launch_project(const double2* Vt, const double2* in, double2* out, const Geo& g, int t, int nev, int nrhs, int mode,
                          double2* coef, long coef_cap, double2* part, long part_cap, hipStream_t s) {
    const long L3 = (long)g.Z * g.Y * g.X, fs = 24L * g.Vh;
    const int ks = project_ks(g, nev);
    // column sets (of four right-hand sides): those whose c fit coef, and of them those per
    // contraction, whose partials fit part (pairs of sets share a wave)
    const long per = 16L * std::max(1, nev), sets = coef_cap / per;
    long psets = ks > 1 ? part_cap / (per * ks) : sets;
    if (psets > 2) psets -= psets & 1;
    if (sets < 1 || psets < 1) return hipErrorInvalidValue;
    const unsigned nrb = (unsigned)((L3 * 3 + 127) / 128);
    const unsigned nfb = (unsigned)((fs + FILL_PER_BLOCK - 1) / FILL_PER_BLOCK);
    // Few modes and right-hand sides on a small timeslice: one launch for c instead of the
    // contraction's two, while a block's passes over its L3 sites stay short.  8 modes, one
    // right-hand side (us per call): 4^3 27 against 32, 600 sites 28 against 33, 12^3 31
    // against 33, 16^3 38 against 34; 64 modes, 64 right-hand sides: 4^3 46 against 49, 600
    // sites 80 against 67.
    const bool direct = L3 <= 2048 && (double)nev * nrhs * L3 * L3 <= (double)(1L << 28);
    // one column set per wave until the waves of 32 rows fill the chip
    const int H = nrhs > 4 && (L3 * 3 + 31) / 32 * ((nrhs + 7) / 8) >= 1024 ? 2 : 1;
    // right-hand sides per apply: fewer than 2^32 threads, pairs of sets together
    const long arhs = ((1L << 24) - 1 - nrb) / (nfb + (nrb + 3) / 4) / 8 * 8;
    for (long r0 = 0; r0 < nrhs; r0 += 4 * sets) {
        const long nr = std::min<long>(4 * sets, nrhs - r0);
        const double2* inr = in + r0 * fs;
        // every c before any output, which may overlap the inputs of other right-hand sides
        if (nev > 0 && direct) {
            hipLaunchKernelGGL(k_proj_coef, dim3(nev, (unsigned)nr), dim3(256), 0, s, Vt, inr, L3, (long)t * L3 * 12, fs, nev, coef);
        } else if (nev > 0) {  // no modes: box(t) = 0 and the apply kernel reads no coefficient
            for (long p0 = 0; p0 < nr; p0 += 4 * psets) {
                ContractArgs a = {};
                a.Vall = Vt; a.f0 = inr + p0 * fs; a.L3 = L3; a.fs = fs;
                a.t0 = a.tv0 = t;
                a.nf = (int)std::min(4 * psets, nr - p0);
                a.nt = 1; a.nev = nev; a.ng = (a.nf + 3) / 4; a.ks = ks;
                a.taup = part;
                const hipError_t e = launch_contract(a, false, false, coef + p0 / 4 * per, s);
                if (e != hipSuccess) return e;
            }
        }
        for (long a0 = 0; a0 < nr; a0 += arhs) {
            const int na = (int)std::min(arhs, nr - a0);
            const unsigned nab = nrb * (unsigned)((na + 4 * H - 1) / (4 * H));
            hipLaunchKernelGGL(H == 2 ? k_proj_apply<2> : k_proj_apply<1>, dim3(nab + nfb * (unsigned)na), dim3(256), 0, s, Vt,
                               inr + a0 * fs, out + (r0 + a0) * fs, L3, fs, t, nev, coef + a0 / 4 * per, na, mode, nab, nrb);
        }
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------- backward of the contractions
//
// Every correlator piece is a sesquilinear form sum <A, M X_t B>_t in the solution
// fields of one source group (four spin-diluted solutions, plus their (1 - box)
// partners for noise).  Its gradient field on timeslice t is therefore
//   grad(t, x) = W1(t) F(t, x) + WP(t) (box(t) F)(t, x),
// with F the group's input fields stacked with their spin components, W1 and WP spin
// matrices that combine the loss weights, Gamma, g5 and the normalisations (the same
// for every group), and box(t) F = sum_k v_k(t) tau_k, tau = V(t)^dag F.  k_tau_weights
// folds WP into tau' = WP tau; k_corr_grad forms W1 F + sum_k v_k tau'_k.

// tau'[grp][ta][k][row] = sum_col WP(t)[row][col] tau_col[k], the columns of a group being
// its sets' 16 columns in turn (noise: phi then phibar).  One thread per (k, row).
template <int N>
__global__ void __launch_bounds__(256) k_tau_weights(const double2* __restrict__ tau, const double2* __restrict__ WP,
                                                     const int* __restrict__ tlist, int nact, int nev, double2* __restrict__ o) {
    const int row = (int)threadIdx.x % N, k = blockIdx.x * (256 / N) + (int)threadIdx.x / N;
    const int ta = blockIdx.y, grp = blockIdx.z;
    if (k >= nev) return;
    const double2* W = WP + ((long)tlist[ta] * N + row) * N;
    double2 v = make_double2(0.0, 0.0);
#pragma unroll
    for (int s = 0; s < N / 16; ++s) {
        const double2* p = tau + ((((long)grp * (N / 16) + s) * nact + ta) * nev + k) * 16;
        for (int c = 0; c < 16; ++c) {
            const double2 w = W[s * 16 + c], x = p[c];
            if (w.x == 0.0 && w.y == 0.0) continue;  // no weight: the column does not enter
            v.x += w.x * x.x - w.y * x.y;
            v.y += w.x * x.y + w.y * x.x;
        }
    }
    o[(((long)grp * nact + ta) * nev + k) * N + row] = v;
}

hipError_t launch_tau_weights(const double2* tau, const double2* WP, const int* tlist, int nact, int nev, int ngrp, bool noise,
                              double2* o, hipStream_t s) {
    if (ngrp <= 0 || nact <= 0) return hipSuccess;
    const int per = noise ? 8 : 16;
    const dim3 grid((nev + per - 1) / per, nact, ngrp);
    if (noise) hipLaunchKernelGGL(k_tau_weights<32>, grid, dim3(256), 0, s, tau, WP, tlist, nact, nev, o);
    else hipLaunchKernelGGL(k_tau_weights<16>, grid, dim3(256), 0, s, tau, WP, tlist, nact, nev, o);
    return hipGetLastError();
}

// Gradient fields of one unit (two distillation groups, or phi and phibar of a noise
// group) on 32 rows (site, colour) of a timeslice per wave: a matrix product over the
// group's (field, spin) inputs, then over the modes, on FP64 matrix instructions.  Rows
// are the A operand (of V: 256 contiguous bytes per mode), the 16 outputs (field, spin)
// of each of the unit's two halves the columns, so V is read once for both halves.
// Bound: the matrix cores and the field streams alike, four waves per SIMD.  At 12^3 x 24 with 21
// modes, 13 distillation and 6 noise groups forward and backward together took 20.9 ms (tau and
// tau' on the host, a VALU kernel here), 2.50 ms with the projections above, 1.80 ms so.
template <bool NOISE>
__global__ void __launch_bounds__(256, 4) k_corr_grad(CorrGradArgs a) {
    constexpr int NIN = NOISE ? 32 : 16;
    const int t = blockIdx.y, unit = blockIdx.z;
    const int g0 = NOISE ? unit : 2 * unit;
    const bool two = NOISE || g0 + 1 < a.ndist;  // a lone group is its own second half, not stored
    const int lane = (int)threadIdx.x & 63, q = lane >> 4, m = lane & 15;
    const long L3 = a.L3, nrow = L3 * 3;
    const long r0 = ((long)blockIdx.x * 4 + (threadIdx.x >> 6)) * 32;
    if (r0 >= nrow) return;  // whole waves
    const int ta = a.tact[t];  // uniform: the timeslice carries weights or not
    const d4 z = {0.0, 0.0, 0.0, 0.0};
    d4 re00 = z, im00 = z, re01 = z, im01 = z, re10 = z, im10 = z, re11 = z, im11 = z;  // half, row tile
    const long tofs = (long)t * L3 * 12;
    if (ta >= 0) {
        // operand rows of this lane (past the last row: the last one, not stored)
        const long row0 = min(r0 + m, nrow - 1), row1 = min(r0 + 16 + m, nrow - 1);
        // W1 F: inputs (field j, spin q)
        const double2* W = (NOISE ? a.W1n : a.W1d) + (long)t * NIN * NIN + (long)m * NIN + q;
        const long f0 = tofs + row0 / 3 * 12 + row0 % 3 + q * 3, f1 = tofs + row1 / 3 * 12 + row1 % 3 + q * 3;
        const long half = two ? 4 * a.fs : 0;
#pragma unroll 1
        for (int j = 0; j < NIN / 4; ++j) {
            const double2* f = (NOISE ? (j < 4 ? a.phi : a.phibar) : a.dist) + ((long)g0 * 4 + (NOISE ? (j & 3) : j)) * a.fs;
            const double2 x0 = f[f0], x1 = f[f1], w0 = W[j * 4];
            mac4(re00, im00, x0, w0);
            mac4(re01, im01, x1, w0);
            if (NOISE) {  // the same inputs, the rows of phibar
                const double2 w1 = W[16 * NIN + j * 4];
                mac4(re10, im10, x0, w1);
                mac4(re11, im11, x1, w1);
            } else {  // the same weights, the second group
                mac4(re10, im10, f[half + f0], w0);
                mac4(re11, im11, f[half + f1], w0);
            }
        }
        // V tau': four modes at a time (past the last: zero)
        const double2* v = a.Vall + ((long)t * a.nev + q) * nrow;
        const double2* tp = NOISE ? a.taun + (((long)g0 * a.nact + ta) * a.nev + q) * 32 + m
                                  : a.taud + (((long)g0 * a.nact + ta) * a.nev + q) * 16 + m;
        const long ts = NOISE ? 16 : (two ? (long)a.nact * a.nev * 16 : 0);
#pragma unroll 1
        for (int k = 0; k < a.nev; k += 4) {
            const bool ok = k + q < a.nev;
            double2 x0 = make_double2(0.0, 0.0), x1 = x0, w0 = x0, w1 = x0;
            if (ok) {
                x0 = v[(long)k * nrow + row0];
                x1 = v[(long)k * nrow + row1];
                w0 = tp[(long)k * NIN];
                w1 = tp[(long)k * NIN + ts];
            }
            mac4(re00, im00, x0, w0);
            mac4(re01, im01, x1, w0);
            mac4(re10, im10, x0, w1);
            mac4(re11, im11, x1, w1);
        }
    }
    // result register i of this lane: row 4 i + q, output m = (field, spin)
    auto store = [&](double2* o, int b, d4 re, d4 im) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const long r = r0 + 16 * b + 4 * i + q;
            if (r < nrow) o[r / 3 * 12 + r % 3] = make_double2(re[i], im[i]);
        }
    };
    const long of = ((long)g0 * 4 + (m >> 2)) * a.fs + tofs + (m & 3) * 3;
    double2* o0 = (NOISE ? a.gphi : a.gdist) + of;
    store(o0, 0, re00, im00);
    store(o0, 1, re01, im01);
    if (two) {
        double2* o1 = NOISE ? a.gphibar + of : o0 + 4 * a.fs;
        store(o1, 0, re10, im10);
        store(o1, 1, re11, im11);
    }
}

hipError_t launch_corr_grad(const CorrGradArgs& a, int T, hipStream_t s) {
    if (2L * a.nnoise + a.ndist > 65535) return hipErrorInvalidValue;  // the callers keep the grids below this
    const unsigned nb = (unsigned)((a.L3 * 3 + 127) / 128);
    if (a.ndist > 0) hipLaunchKernelGGL(k_corr_grad<false>, dim3(nb, T, (a.ndist + 1) / 2), dim3(256), 0, s, a);
    if (a.nnoise > 0) hipLaunchKernelGGL(k_corr_grad<true>, dim3(nb, T, a.nnoise), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace dlma
