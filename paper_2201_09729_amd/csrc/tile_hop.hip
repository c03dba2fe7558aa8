// Schur stencils on right-hand-side tiles (tile.h): matrix products of link entries and
// neighbour spinors on the bfloat16 matrix instructions.
//
// With Gamma_d = 1 -+ g_mu and U'_d the matrix acting on neighbour d (8 of them),
//   (H psi)(x)_{s' a} = sum_d sum_{s b} (Gamma_d)_{s' s} (U'_d)_{ab} psi_d{s b}.
// A wave owns one output site at a time.  Operand A: lane (row, s) of a 16-row tile holds
// row (s', a, re or im) of input spin s: three complex entries per direction, each the
// link word turned by the lane's coefficient in {0, +-1, +-i} (the four turned forms of a
// site's words are in LDS, a lane reads the one it needs).  Rows 4 s' + i: tile 0 colours 0 and 1 (re, im each), tile 1
// colour 2, two rows empty.  Operand B is the field itself.  Eight directions of three
// words fill six instructions of K = 32 per row tile.  The result lane (q, n) then holds
// the six reals of spin q of right-hand side n: the layout that is stored, and an operand
// again for the clover block of K1 (its FP32 values split into three bfloat16 terms, exact to
// 2^-24).
//   K1 (odd):  out = C (ch H in), ch = -1/2;  K2 (even): out = C x + 1/2 H in,
// K2's own-site term being a ninth direction of the same product.
// Block order: an XCD owns a contiguous range of timeslices (and of z, with few timeslices)
// and walks strips of y rows outermost, then z, then its timeslices, so the +-t and +-z
// neighbours of a strip stay in its L2.
// Bound: the texture address path (0.74 to 0.87 busy), L2 misses (hits 0.59 to 0.64; the fields
// come 1.6 to 2 times over from the memory side) and LDS (the turned words are read a word per
// lane, bank conflicts in 0.34 to 0.40 of the cycles), in three uneven configurations with 160
// right-hand sides.  Waves per SIMD by registers: K1 six (78), K2 with (rh, v) five (91), K2 with
// (t, s) four (100).  48x24^3 with 96 right-hand sides: K1 1.29, K2 1.44 ms (1.9 and 2.1 ms with
// one thread per site and one to four right-hand sides, FP32 arithmetic on the vector units);
// 24x12^3 with 72: 74 and 71 us (94 and 98).  Blocks of two to six tiles sharing a site's turned
// words were slower (1.45 to 1.8 ms): the registers they need leave three waves per SIMD.
#include "tile_dev.h"

namespace dlma {

// Which turned form of a link word a lane of operand A takes: entry [d][lane], d = 2 mu +
// backward; d = 8: the identity within a chirality (clover).  A word u = (ur, ui) of a
// matrix enters row "re" as (Re z, -Im z) and row "im" as (Im z, Re z), z = i^k u; these
// are four forms: 0 (ur, -ui), 1 (ui, ur), 2 (-ur, ui), 3 (-ui, -ur), and 4 zero.
struct FormTable { uint8_t f[9][64]; };
constexpr FormTable make_forms() {
    FormTable t{};
    // g_mu entries (row s', partner column, code) in the chiral basis; codes 1: +1 2: -1 3: +i 4: -i
    constexpr int col[4][4] = {{2, 3, 0, 1}, {3, 2, 1, 0}, {3, 2, 1, 0}, {2, 3, 0, 1}};
    constexpr int gam[4][4] = {{2, 2, 2, 2}, {4, 4, 3, 3}, {2, 1, 1, 2}, {4, 3, 3, 4}};
    constexpr uint8_t re[5] = {4, 0, 2, 3, 1}, im[5] = {4, 1, 3, 0, 2};
    constexpr int neg[5] = {0, 2, 1, 4, 3};
    for (int d = 0; d < 9; ++d)
        for (int l = 0; l < 64; ++l) {
            const int s = l >> 4, sp = (l & 15) >> 2;
            int code = 0;
            if (d == 8) {
                code = (s >> 1) == (sp >> 1) ? 1 : 0;
            } else {
                const int mu = d >> 1;
                if (s == sp) code = 1;
                else if (col[mu][sp] == s) code = (d & 1) ? gam[mu][sp] : neg[gam[mu][sp]];  // 1 + g backward, 1 - g forward
            }
            t.f[d][l] = (l & 1) ? im[code] : re[code];
        }
    return t;
}
__device__ const FormTable k_forms = make_forms();

__device__ __forceinline__ u32x4 quad(const uint32_t* w, int i) { return (u32x4){w[i], w[i + 1], w[i + 2], w[i + 3]}; }

constexpr int TILE_NW = 4;  // waves per block; left to itself the compiler moves values through AGPRs (K1 +3%)

template <int KIND, int FL>
__global__ void __launch_bounds__(TILE_NW * 64) __attribute__((amdgpu_waves_per_eu(3)))
k_tile_hop(const TileHopJob* __restrict__ jobs, int njob, int tw0, int twn) {
    constexpr int NQ = hop_nq(FL);
    constexpr bool DOTS = NQ > 0;
    const int bid = blockIdx.x;
    int jb = 0;
    while (jb + 1 < njob && bid >= jobs[jb + 1].blk0) ++jb;
    const TileHopJob& J = jobs[jb];
    // block -> (tile, strip, z, timeslice)
    const int lb = bid - J.blk0, xcd = lb & 7, k0 = lb >> 3;
    const int T = J.g.T, Tw = twn > 0 ? twn : T;
    const int nT = tile_xcd_t(Tw), nZ = 8 / nT, xt = xcd % nT, xz = xcd / nT;
    const int tl = xt * Tw / nT, nt = (xt + 1) * Tw / nT - tl;
    const int zl = xz * J.g.Z / nZ, nz = (xz + 1) * J.g.Z / nZ - zl;
    const int per = J.nstrip * nz * nt;
    if (per == 0) return;
    const int tile = k0 / per;
    if (tile >= J.ntile) return;
    const int kk = k0 - tile * per, sz = kk / nt;
    const int strip = sz / nz, z = zl + sz - strip * nz;
    const int tw = tl + (kk - sz * nt);
    const int t = twn > 0 ? (tw0 + tw < T ? tw0 + tw : tw0 + tw - T) : tw;
    const int Y = J.g.Y, Xh = J.g.Xh, Vh = J.g.Vh;
    const int y0 = strip * J.R, ns = min(J.R, Y - y0) * Xh;
    const int cb0 = ((t * J.g.Z + z) * Y + y0) * Xh;
    const int sb = t * J.nbt + z * J.nstrip + strip;

    const int lane = (int)threadIdx.x & 63, q = lane >> 4, n = lane & 15;
    const int wave = wave_uniform((int)threadIdx.x >> 6);
    const int r = tile * TILE + n;
    const bool use = r < J.nrhs && (J.active == nullptr || J.active[r] != 0);  // still iterating
    if (__ballot(use) == 0) {  // nothing to do: zero partials
        if (DOTS && (int)threadIdx.x < 16 * NQ) {
            const int c = (int)threadIdx.x & 15, k = (int)threadIdx.x >> 4;
            if (tile * TILE + c < J.nrhs) J.part[((size_t)(tile * TILE + c) * NQ + k) * J.pstride + sb] = 0.0;
        }
        return;
    }
    __shared__ uint32_t lds_links[TILE_NW * 720];
    const uint32_t lane12 = 12u * (uint32_t)lane;
    const uint32_t row0 = (uint32_t)((lane >> 1) & 1);  // colour of this lane's row in tile 0
    const bool upper = (lane & 2) == 0;                  // tile 1 holds rows i = 0, 1 only
    // this lane's clover row (s' % 2, colour) and columns (s % 2, .) in words
    const uint32_t sp = (uint32_t)((lane & 15) >> 2);
    const uint32_t crow = ((sp >> 1) * 6u + (sp & 1u) * 3u) * 6u + (uint32_t)(q & 1) * 3u;
    // this lane's place in the turned words of its rows (tile 1's empty rows: zeros)
    uint32_t at[8];
#pragma unroll
    for (int d = 0; d < 8; ++d) at[d] = (uint32_t)k_forms.f[d][lane] * 144u;
    const uint32_t atc = (uint32_t)k_forms.f[8][lane] * 144u;
    const WSrc L = wsrc(J.L, 576u * (uint32_t)Vh);
    const WSrc RH = DOTS ? wsrc(J.rh, 48u * (uint32_t)Vh) : L;
    const WSrc in = tile_src(J.in, Vh, tile), out = tile_src(J.out, Vh, tile);
    const WSrc xs = tile_src(KIND == K2 ? J.x : J.in, Vh, tile);
    uint32_t* lw = &lds_links[wave * 720];
    for (int e = lane; e < 144; e += 64) lw[576 + e] = 0;
    // offsets to the neighbours in t and z, the same for every site of the block
    const int sZ = Y * Xh, sT = J.g.Z * sZ;
    const int dtp = (t + 1 == T ? 1 - T : 1) * sT, dtm = (t == 0 ? T - 1 : -1) * sT;
    const int dzp = (z + 1 == J.g.Z ? 1 - J.g.Z : 1) * sZ, dzm = (z == 0 ? J.g.Z - 1 : -1) * sZ;
    double qs[NQ > 0 ? NQ : 1];
#pragma unroll
    for (int k = 0; k < NQ; ++k) qs[k] = 0.0;

    // a site's links and clover (144 words) come with one load of 48 lanes, the next site's
    // while this one is worked on
    u32x3 next = {0, 0, 0};
    if (lane < 48 && wave < ns) next = wld3(L, lane12, 576u * (uint32_t)(cb0 + wave));
    for (int i = wave; i < ns; i += TILE_NW) {
        const int cb = cb0 + i;
        int nb[8];
        {
            const int row = (int)mdiv(i, J.g.mXh), xh = i - row * Xh, y = y0 + row;
            const int odd = (t + z + y + J.par) & 1;
            const int xf = xh + odd, xb = xh + odd - 1;
            nb[0] = cb + dtp;
            nb[1] = cb + dtm;
            nb[2] = cb - xh + (xf == Xh ? 0 : xf);
            nb[3] = cb - xh + (xb < 0 ? Xh - 1 : xb);
            nb[4] = cb + (y + 1 == Y ? 1 - Y : 1) * Xh;
            nb[5] = cb + (y == 0 ? Y - 1 : -1) * Xh;
            nb[6] = cb + dzp;
            nb[7] = cb + dzm;
        }
        // every load first: eight neighbours, the own site
        u32x3 w[8], own = {0, 0, 0}, rw = {0, 0, 0};
#pragma unroll
        for (int d = 0; d < 8; ++d) w[d] = wld3(in, lane12, 768u * (uint32_t)nb[d]);
        if (KIND == K2) own = wld3c<CP_NT>(xs, lane12, 768u * (uint32_t)cb);
        if (DOTS) rw = wld3(RH, 12u * (uint32_t)q, 48u * (uint32_t)cb);
        // the four turned forms of the site's words
        if (lane < 48) {
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                const uint32_t u = next[e], v = (u >> 16) | (u << 16);
                lw[3 * lane + e] = u ^ 0x80000000u;
                lw[144 + 3 * lane + e] = v;
                lw[288 + 3 * lane + e] = u ^ 0x00008000u;
                lw[432 + 3 * lane + e] = v ^ 0x80008000u;
            }
            if (i + TILE_NW < ns) next = wld3(L, lane12, 576u * (uint32_t)(cb + TILE_NW));
        }
        __builtin_amdgcn_wave_barrier();
        uint32_t A0[28], A1[28], c0[3], c1[3], B[28];
#pragma unroll
        for (int d = 0; d < 8; ++d)
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                A0[3 * d + e] = lw[at[d] + 3 * row0 + 9 * d + e];
                A1[3 * d + e] = lw[(upper ? at[d] : 576u) + 9 * d + 6 + e];
                B[3 * d + e] = w[d][e];
            }
#pragma unroll
        for (int e = 0; e < 3; ++e) {
            c0[e] = lw[atc + crow + 6 * row0 + 72 + e];
            c1[e] = lw[(upper ? atc : 576u) + crow + 84 + e];
            A0[24 + e] = c0[e];
            A1[24 + e] = c1[e];
        }
        A0[27] = A1[27] = B[27] = 0;
        f32x4 r0 = {0, 0, 0, 0}, r1 = {0, 0, 0, 0};
#pragma unroll
        for (int j = 0; j < 6; ++j) {
            r0 = mma16(quad(A0, 4 * j), quad(B, 4 * j), r0);
            r1 = mma16(quad(A1, 4 * j), quad(B, 4 * j), r1);
        }
        if (KIND == K2) {  // H in enters with 1/2, C x with 1
            r0 *= 0.5f;
            r1 *= 0.5f;
            const u32x4 b = {own.x, own.y, own.z, 0};
            r0 = mma16(quad(A0, 24), b, r0);
            r1 = mma16(quad(A1, 24), b, r1);
        } else {
            // C acts on the FP32 sums, split into three bfloat16 terms of the operand's layout
            float v[6] = {r0[0], r0[1], r0[2], r0[3], r1[0], r1[1]};
            uint32_t tt[12], a0[12], a1[12];
#pragma unroll
            for (int s = 0; s < 3; ++s)
#pragma unroll
                for (int e = 0; e < 3; ++e) {
                    const uint32_t x = pack16(v[2 * e], v[2 * e + 1]);
                    v[2 * e] -= word_lo(x);
                    v[2 * e + 1] -= word_hi(x);
                    tt[3 * s + e] = x;
                    a0[3 * s + e] = c0[e];
                    a1[3 * s + e] = c1[e];
                }
#pragma unroll
            for (int e = 9; e < 12; ++e) tt[e] = a0[e] = a1[e] = 0;
            r0 = r1 = (f32x4){0, 0, 0, 0};
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                r0 = mma16(quad(a0, 4 * j), quad(tt, 4 * j), r0);
                r1 = mma16(quad(a1, 4 * j), quad(tt, 4 * j), r1);
            }
        }
        // result: K1 times ch = -1/2
        float v[6] = {r0[0], r0[1], r0[2], r0[3], r1[0], r1[1]};
        uint32_t ow[3];
#pragma unroll
        for (int e = 0; e < 6; ++e)
            if (KIND == K1) v[e] *= -0.5f;
#pragma unroll
        for (int e = 0; e < 3; ++e) ow[e] = pack16(v[2 * e], v[2 * e + 1]);
        if (use) {
            wide_store_begin();
            wst3<CP_NT>(out, lane12, 768u * (uint32_t)cb, (u32x3){ow[0], ow[1], ow[2]});
            wide_store_end();
        }
        if (DOTS) {
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                const uint32_t hw = rw[e], xw = own[e];
                const double vr = v[2 * e], vi = v[2 * e + 1], ar = word_lo(hw), ai = word_hi(hw);
                if (FL & F_DOTX) {  // conj(out) x, |out|^2, and conj(rh) out of the stored out
                    const double xr = word_lo(xw), xi = word_hi(xw), sr = word_lo(ow[e]), si = word_hi(ow[e]);
                    qs[0] += vr * xr + vi * xi;
                    qs[1 < NQ ? 1 : 0] += vr * xi - vi * xr;
                    qs[2 < NQ ? 2 : 0] += vr * vr + vi * vi;
                    qs[3 < NQ ? 3 : 0] += ar * sr + ai * si;
                    qs[4 < NQ ? 4 : 0] += ar * si - ai * sr;
                } else {  // conj(rh) out
                    qs[0] += ar * vr + ai * vi;
                    qs[1 < NQ ? 1 : 0] += ar * vi - ai * vr;
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    if (DOTS) {
        __shared__ double sums[TILE_NW][NQ > 0 ? NQ : 1][16];
#pragma unroll
        for (int k = 0; k < NQ; ++k) {
            const double v = sum_over_q(use ? qs[k] : 0.0);
            if (q == 0) sums[wave][k][n] = v;
        }
        __syncthreads();
        if ((int)threadIdx.x < 16 * NQ) {
            const int c = (int)threadIdx.x & 15, k = (int)threadIdx.x >> 4;
            if (tile * TILE + c < J.nrhs)
                J.part[((size_t)(tile * TILE + c) * NQ + k) * J.pstride + sb] = ((sums[0][k][c] + sums[1][k][c]) + sums[2][k][c]) + sums[3][k][c];
        }
    }
}

hipError_t launch_tile_hop(int kind, int flags, const TileHopJob* d, int njob, int nblocks, int tw0, int twn,
                           hipStream_t s) {
    if (nblocks <= 0) return hipSuccess;
    const dim3 grid(nblocks), block(TILE_NW * 64);
#define DLMA_TILE_CASE(KIND, FL)                                                                          \
    if (kind == (KIND) && flags == (FL)) {                                                                \
        hipLaunchKernelGGL((k_tile_hop<KIND, (FL)>), grid, block, 0, s, d, njob, tw0, twn);             \
        return hipGetLastError();                                                                         \
    }
    DLMA_TILE_CASE(K1, 0)
    DLMA_TILE_CASE(K2, 0)
    DLMA_TILE_CASE(K2, F_DOTR)
    DLMA_TILE_CASE(K2, F_DOTX | F_DOTXH)
    return hipErrorInvalidValue;
}

}  // namespace dlma
