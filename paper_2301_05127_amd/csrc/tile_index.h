// Index arithmetic of the tile passes (tile.hip), usable from host code so that a CPU
// check can enumerate every index the kernels form.
#pragma once

#if !defined(LOSS_HD)
#if defined(__HIPCC__)
#define LOSS_HD __host__ __device__ inline
#else
#define LOSS_HD inline
#endif
#endif

namespace loss {

constexpr int kTileM = 64;        // intervals of a piece, at most
constexpr int kTileC = 8;         // rows per wave
constexpr int kTileWaves = kTileM / kTileC;
constexpr int kTileHalo = 20;     // taps on either side of a junction, at most
constexpr int kTapW = 2 * kTileHalo + 1;
// LDS row of the x solve: kTileHalo nodes left of the piece, its own nodes (and, where it
// has fewer than kTileM, the closing node), then the closing node and the taps right of it
constexpr int kRowOwn = kTileHalo;
constexpr int kRowRight = kRowOwn + kTileM;
constexpr int kRowPitch = 112;    // = 48 mod 64: the four rows a wave solves at once start in different banks

// a cut lies this far inside a patch: its row's weights beyond the patch ends are then below
// 0.268^16 = 7e-10 of the others (FP32 rounding: 6e-8)
constexpr int kCutGap = 16;
constexpr int kTileIn = 3;        // junctions inside a piece, at most
constexpr int kTileInGap = 8;     // nodes between them, at least: one per chunk of rows, one per lane

// Window of one piece along an axis: nodes s .. e, hl nodes left of s and hr nodes right
// of e that the taps of its junctions (the two ends and up to kTileIn inside) reach.
struct Piece {
    int s, e, m;       // m = e - s
    int hs, he;        // taps on either side of the junction rows s and e (0: natural end)
    int hl, hr;
    int ni, hi;        // junctions inside, taps on either side of them
};

// as the tables hold it: {s, e, hs | he << 8 | hl << 16 | hr << 24, ni | hi << 8}
LOSS_HD Piece make_piece(int s, int e, int z, int w)
{
    Piece p;
    p.s = s;
    p.e = e;
    p.m = e - s;
    p.hs = z & 255;
    p.he = (z >> 8) & 255;
    p.hl = (z >> 16) & 255;
    p.hr = (z >> 24) & 255;
    p.ni = w & 255;
    p.hi = w >> 8;
    return p;
}

// halo entries of a piece: i < hl is node s - hl + i, the others node e + (i - hl)
LOSS_HD int halo_count(const Piece &p) { return p.hl + p.hr + 1; }
LOSS_HD int halo_pos(const Piece &p, int i) { return i < p.hl ? p.s - p.hl + i : p.e + (i - p.hl); }
// their places in the LDS row of the x solve
LOSS_HD int halo_slot(const Piece &p, int i) { return i < p.hl ? kRowOwn - p.hl + i : kRowRight + (i - p.hl); }
// place of the node d after the start of the piece, as a tap reads it
LOSS_HD int tap_slot(const Piece &p, int d) { return d < p.m ? kRowOwn + d : kRowRight + (d - p.m); }

// the grid node of position k of a line: wrapped on a periodic axis (node N is node 0),
// else clamped (taps outside the line carry a zero coefficient)
LOSS_HD int line_node(int k, int N, int periodic)
{
    if (periodic) return k < 0 ? k + N : (k >= N ? k - N : k);
    return k < 0 ? 0 : (k > N ? N : k);
}

}  // namespace loss
