// Right-hand-side tiles: the layout, jobs and launchers of the BF16 inner solver (BiCGStab)
// for many right-hand sides.
//
// Sixteen right-hand sides of one site are the columns of a matrix product: the hopping
// term of an output site is a (24 x 192)-matrix of link entries times the (192 x 16)
// spinor components of its eight neighbours, which is what the matrix instructions take
// (v_mfma_f32_16x16x32: operand lane l holds row or column l % 16 at eight consecutive
// 16-bit values of group l / 16; result register i of lane l is row 4 (l / 16) + i of
// column l % 16).  A field is stored so that its words are that operand:
//   [tile][Vh][spin 4][rhs 16][colour 3], one complex number (two bfloat16) per word
// Lane (q, n) = (l / 16, l % 16) of a wave holds spin q of right-hand side n: 12 bytes,
// 768 contiguous bytes per site and wave.
//   links   [Vh][144] words per output parity: [direction 8][row 3][col 3], the matrices that
//           act on the neighbours (forward mu: U_mu(x); backward: U_mu(x - mu)^dag), direction
//           2 mu + backward; then the clover term (A_ee or A_oo^-1), [block 2][row 6][col 6]
//   shadow residual [Vh][spin 4][colour 3] words, shared by every right-hand side
#pragma once
#include "kernels.h"

namespace dlma {

constexpr int TILE = 16;         // right-hand sides per tile
constexpr int TCONV_SITES = 32;  // sites per block of the layout conversions

inline int tile_count(int nrhs) { return (nrhs + TILE - 1) / TILE; }
// Sites per block of the stencil (about) and vector kernels, whose four waves take them in
// turn: enough to spread a block's start, few while the blocks do not fill the chip.  Vector
// kernels, 8x12x10x12 with 16 right-hand sides: the x, r, p update 24 us with 64 sites per block.
// Stencils, whole BF16 solves (ms) with 8 and 48 sites per block: 24x8x12x16 with 16 right-hand
// sides (18432 tile sites) 8.6, 9.0; 10x12x10x12 with 44 (21600) 9.5, 10.1; 12x8x16x10 with 48
// (23040) 10.8, 10.2; 16x12^3 with 32 (27648) 11.4, 10.8; 24x12^3 with 48 (62208) 22.6, 20.5.
// 48x24^3 with 96: 24 to 100 sites of a stencil block are alike, 256 are 10% slower.
inline long tile_sites(int Vh, int nrhs) { return (long)Vh * tile_count(nrhs); }
inline int tile_hop_sites(int Vh, int nrhs) { return tile_sites(Vh, nrhs) < 22000 ? 8 : 48; }
inline int tile_vec_sites(int Vh, int nrhs) { return tile_sites(Vh, nrhs) < 65536 ? 8 : 64; }

// One Schur stencil of one configuration.  A block covers R y rows (the last strip fewer) of
// one z plane of one timeslice, for one tile.
struct TileHopJob {
    Geo g;
    int par, nrhs, ntile;
    int R, nstrip, nbt;    // y rows per block, strips per plane, blocks per timeslice = Z * nstrip
    int blk0;
    const uint32_t* L;     // links and clover
    uint32_t *in, *x, *out;
    uint32_t* rh;          // shadow residual
    const int* active;     // [nrhs] or nullptr
    double* part;          // part[(r * NQ + q) * pstride + site block]
    int pstride;           // T * nbt
};
// equal strips: 20x12x10x12 with 32 right-hand sides 11.8 ms per solve with strips of 8 and 2
// rows, 11.5 with 5 and 5
inline int tile_hop_rows(const Geo& g, int nrhs) {
    const int r = tile_hop_sites(g.Vh, nrhs) / g.Xh;
    if (r < 1) return 1;
    const int n = (g.Y + r - 1) / r;
    return (g.Y + n - 1) / n;
}
inline int tile_hop_nbt(const Geo& g, int nrhs) { const int r = tile_hop_rows(g, nrhs); return g.Z * ((g.Y + r - 1) / r); }
// XCDs along the timeslices of a launch (the rest along z): all eight where they divide the
// timeslices or leave few idle, else the largest power of two that does
HD int tile_xcd_t(int Tw) {
    int n = 8;
    while (n > 1 && Tw % n != 0 && Tw < 4 * n) n >>= 1;
    return n;
}
// blocks of a launch of one job over twn timeslices (twn = T: all of them)
inline int tile_hop_blocks(const TileHopJob& j, int twn) {
    const int nT = tile_xcd_t(twn), nZ = 8 / nT;
    return 8 * ((twn + nT - 1) / nT) * ((j.g.Z + nZ - 1) / nZ) * j.nstrip * j.ntile;
}

// kind, flags as hop.h (K1 0; K2 0, F_DOTR, F_DOTX | F_DOTXH); tw0, twn as HopCfg
hipError_t launch_tile_hop(int kind, int flags, const TileHopJob* d, int njob, int nblocks, int tw0, int twn,
                           hipStream_t s);

// Steps of one iteration (BiVecMode BV_RR, BV_SH, BV_XRP) on tile fields
struct TileVecJob {
    int Vh, nrhs, ntile, nsb, blk0;  // nsb = ceil(Vh / sites); blocks = nsb * ntile
    int sites;                       // per block
    uint32_t *r, *rh, *p, *v, *s, *t, *x;
    const double2 *alpha, *omega, *beta;
    const int* active;
    double *part, *part_s;
    int pstride;
    const int *tdist, *titer;  // reach of the first pass (in_reach) or nullptr
    int vt, T;
};
hipError_t launch_tile_vec(const TileVecJob* d, int njob, int nblocks, int mode, hipStream_t s);

// FP64 Schur source <-> tiles.  Conversion in: a = b = P(src / |src|), c = 0 (VecJob's
// k_conv_from64), partials of |a|^2; out: the tile field as a field of the [rhs] layouts.
struct TileConvJob {
    int Vh, nrhs, ntile, nsb, blk0;  // nsb = ceil(Vh / TCONV_SITES); blocks = nsb * ntile
    SF<P64> src;
    const double* s;   // [nrhs] |src|^2
    const int* active; // [nrhs]: the others keep their fields
    uint32_t *a, *b, *c;
    double* part;
    int pstride;
    const int* tsup;   // the source vanishes where t - tdil .. t + tdil are unflagged (VecJob)
    int tdil, vt, T;
};
hipError_t launch_tile_conv(const TileConvJob* d, int njob, int nblocks, hipStream_t s);
struct TileBackJob {
    int Vh, nrhs, ntile, nsb, blk0;
    uint32_t *a;
    uint32_t* v;  // [rhs][12][Vh]
};
hipError_t launch_tile_back(const TileBackJob* d, int njob, int nblocks, hipStream_t s);

// the links, and the clover words, of one output parity from the FP64 planes; the random
// shadow residual
hipError_t launch_tile_links(const double2* U64, const Geo& g, int par, uint32_t* L, hipStream_t s);
hipError_t launch_tile_clover(const double2* C64, int Vh, uint32_t* L, hipStream_t s);
hipError_t launch_tile_random(uint32_t* f, int Vh, unsigned seed, hipStream_t s);

}  // namespace dlma
