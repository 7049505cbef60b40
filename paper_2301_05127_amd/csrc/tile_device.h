// Device building blocks of the tile passes (tile.hip) and of the single-axis passes built
// the same way (tile_axis.hip): node access through buffer descriptors, the solve along the
// rows by chunks whose carries are sums with tabulated coefficients, and the solve of a row
// of x by 16 lanes.  OP is one of TileOp: slopes, moments, transposed slopes.
#pragma once

#include <hip/hip_runtime.h>

#include "line_device.h"
#include "loss_internal.h"
#include "tile_index.h"

namespace loss {

namespace {

// Where the tile lives: element of node (0, 0) of its plane in a field (of its shot) and in
// a media array (uniform), the lane's column (clamped into the piece) and its byte offset,
// whether the lane owns a node, the bytes per row.
struct Place {
    int64_t fb, mb;
    int shot, o;
    int xc;
    bool act;
    unsigned vx, rs4;
};

// Node access through buffer descriptors: scalar base, scalar row offset, the lane's column
// offset: one instruction and no address arithmetic per access, and one register for the
// addresses of every row and array (64-bit addresses formed per access were half of the
// kernels' vector instructions).  Offsets are 32-bit bytes: a field of one shot stays below
// 2^30 elements.
typedef __amdgpu_buffer_rsrc_t Buf;
__device__ __forceinline__ Buf buf(const float *p)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p), 0, -1, 0x00020000);
}
__device__ __forceinline__ float ld(Buf b, unsigned row, unsigned col)
{
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(b, (int)col, (int)row, 0));
}
__device__ __forceinline__ void st(Buf b, unsigned row, unsigned col, float v)
{
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), b, (int)col, (int)row, 0);
}

// Workgroups are dealt round-robin to the 8 XCDs; each XCD gets runs of `chunk` tiles (x
// fastest), so that neighbours' halos meet in one L2.  One run per XCD, except where elastic
// tiles are few (they are in flight at nearly the same time: runs of whole rows, about 16
// tiles, keep the XCDs' reads close together) and for the z derivatives (of 257^3 x 2 205 / 200
// us a kernel).  Measured, one run per XCD / runs of 16: elastic us per step 65^3 (260 tiles)
// 48.4 / 46.5, 193^3 (2316) 393 / 386, 225^3 (3600) 583 / 575, 257 x 257 x 201 (4020) 706 / 695,
// 257^3 (5140) 842 / 840, x 2 (10 280) 1617 / 1641, 225^3 x 2 (7200) 1118 / 1127; acoustic 16 x
// 1101 x 706 with layers 7.65 / 8.17 ms a pass.  Shots of one tile next to each other (the media
// read once) lose: 64 x 1025^2 382 -> 410 us a kernel.
// A single axis: runs of 16 where a field's columns are many.  Second derivatives along z of
// 2 x 257^3 (1032 column groups) 77 / 71 us; of 2 to 100 groups within 2 % either way, 128
// groups 60 / 55, 200 groups 61 / 63, 400 and 1000 the same.
constexpr int kXcdChunk = 16;

__device__ __forceinline__ int xcd_range() { return (int)((blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3)); }
__device__ __forceinline__ int xcd_order(int chunk)
{
    const int i = (int)(blockIdx.x >> 3), r = i / chunk;
    return (r * 8 + (int)(blockIdx.x & 7)) * chunk + (i - r * chunk);
}

// workgroups of a launch: whole rounds of 8 chunks, those past the last tile return
inline int64_t xcd_blocks(int64_t nreal, int chunk) { return (nreal + 8 * (int64_t)chunk - 1) / (8 * (int64_t)chunk) * 8 * chunk; }

constexpr int kHaloPre = 4;     // halo rows per wave and field loaded ahead of the solve

// orders the LDS accesses of a wave's lanes among each other (the wave runs in lockstep;
// this keeps the compiler from moving them across)
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// sum over the 16 lanes of a DPP row, in every lane
__device__ __forceinline__ float row_sum(float v)
{
    auto ror = [](float x, auto dc) {
        constexpr int D = decltype(dc)::value;
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x120 + D, 0xF, 0xF, true));
    };
    v += ror(v, std::integral_constant<int, 8>{});
    v += ror(v, std::integral_constant<int, 4>{});
    v += ror(v, std::integral_constant<int, 2>{});
    v += ror(v, std::integral_constant<int, 1>{});
    return v;
}

__device__ __forceinline__ Piece piece_of(const TileAxis &t, int i)
{
    const int4 p = t.piece[i];
    return make_piece(p.x, p.y, p.z, p.w);
}

// ---- rows ------------------------------------------------------------------------
// One wave's chunk of one field: rows q .. q + 7 of a piece, u[0 .. 9] = rows q - 1 .. q + 8.

// right-hand side of row c before its weight sc
template <int OP>
__device__ __forceinline__ float row_rhs(const float (&u)[kTileC + 2], int c)
{
    if constexpr (OP == TILE_D1) return u[c + 2] - u[c];
    else if constexpr (OP == TILE_D2) return (u[c + 2] - u[c + 1]) - (u[c + 1] - u[c]);
    else return u[c + 1];
}

// Taps along x on differences from the junction's own value (see taps_own): those of single axes
// (ALONE), slopes but for pieces with junctions inside, where registers are short, and moments.
template <int OP, bool IN, bool ALONE>
constexpr bool kDiffX = OP == TILE_D2 || (OP == TILE_D1 && !IN && ALONE);

// In both sweeps of a solve the product that is rounded by itself is the one with the
// neighbouring row, 0.27 of the sum; the other one is up to 1.3 times it.  (The other way
// round, slopes along the rows of white noise were 1.04 times as far from 64 bits as those of
// the passes along one axis, now 0.94, along x 0.96 -> 0.88, of smooth fields 0.96-1.22 ->
// 0.8-0.95; as many instructions, the same time.)
__device__ __forceinline__ float sweep(float a, float own, float f, float next) { return fmaf(a, own, f * next); }

// The rows' eliminated values from a zero carry (transposed: their right-hand sides, see
// rows_finish), B and W of the chunk.
template <int OP>
__device__ __forceinline__ void rows_local(const TileChunk &t, const float (&u)[kTileC + 2], float (&y)[kTileC],
                                           float &B, float &W, float s3)
{
    float z[kTileC], v = 0.f;
#pragma unroll
    for (int c = 0; c < kTileC; ++c) {
        if constexpr (OP == TILE_DT) {
            y[c] = t.sc[c] * u[c + 1];          // weights of 1 and 0
            v = sweep(s3, y[c], t.nf[c], v);
        } else {
            v = sweep(t.sc[c], row_rhs<OP>(u, c), t.nf[c], v);
            y[c] = v;
        }
        z[c] = v;
    }
    B = v;
    v = 0.f;
#pragma unroll
    for (int c = kTileC - 1; c >= 0; --c) v = sweep(t.fi[c], z[c], t.g[c], v);
    W = v;
}

// IN: pieces may hold junctions inside.  Kernels of their own: the junctions' sums take
// registers that the elastic kernels do not have to spare.

// Shares of the tap sums: of the start, of the closing right-hand side, of the junctions inside.
struct Taps {
    float s = 0.f, e = 0.f, j[kTileIn] = {};
    float l = 0.f;              // transposed: the taps left of the piece of its start alone
};

// from a wave's own rows.  Single axes take slopes and moments of the differences from the
// junction's own value (us, ue), whose share is added once: the taps cancel to a difference of
// the field, and of the values themselves the rounding of the products would remain.  The tile
// kernels take the values (us = ue = 0): two more loads a field cost them 1-4 %, and their
// junctions round as those of the passes along one axis do
template <int OP, bool IN>
__device__ __forceinline__ void taps_own(const TileChunk &t, const float (&u)[kTileC + 2], float us, float ue, Taps &p)
{
    if (t.any_ts != 0.f) {          // uniform
#pragma unroll
        for (int c = kTileC - 1; c >= 0; --c) p.s = fmaf(t.ts[c], u[c + 1] - us, p.s);   // the nearest last
    }
    if (t.any_te != 0.f) {
#pragma unroll
        for (int c = 0; c < kTileC; ++c) p.e = fmaf(t.te[c], u[c + 1] - ue, p.e);
    }
    if (IN && t.any_in) {
#pragma unroll
        for (int j = 0; j < kTileIn; ++j)
#pragma unroll
            for (int c = 0; c < kTileC; ++c) p.j[j] = fmaf(t.tj[j][c], u[c + 1], p.j[j]);
    }
}

// from halo entry i of value v
template <int OP, bool IN>
__device__ __forceinline__ void taps_halo(const Piece &pc, const float4 *hc, int i, float v, float us, float ue, Taps &p)
{
    const float4 c = hc[i];
    p.s = fmaf(c.x, v - us, p.s);
    p.e = fmaf(c.y, v - ue, p.e);
    if (IN && pc.ni > 0) {   // uniform
        p.j[0] = fmaf(c.z, v, p.j[0]);
        const float w = c.w * v;        // of the last one, when there are several
#pragma unroll
        for (int j = 1; j < kTileIn; ++j) p.j[j] += j == pc.ni - 1 ? w : 0.f;
    }
    if (OP == TILE_DT && i < pc.hl) p.l = fmaf(c.x, v, p.l);
}

// A wave publishes B, W and its shares of each field into its own row buffer once its x solves
// are done: kPublish floats per field.
constexpr int kWaveLds = kTileC * kRowPitch;
template <int OP, bool IN>
constexpr int kPublish = 256 + (IN ? 64 * kTileIn : 0) + (OP == TILE_DT ? 64 : 0);

template <int OP, bool IN>
__device__ __forceinline__ void rows_publish(const Piece &pc, float *ex, int lane, float B, float W, const Taps &p)
{
    ex[lane] = B;
    ex[64 + lane] = W;
    ex[128 + lane] = p.s;
    ex[192 + lane] = p.e;
    if (IN && pc.ni > 0) {   // uniform
#pragma unroll
        for (int j = 0; j < kTileIn; ++j) ex[256 + 64 * j + lane] = p.j[j];
    }
    if (OP == TILE_DT) ex[kPublish<OP, IN> - 64 + lane] = p.l;
}

// The chunk's rows from its carries; returns the carry from below (the value at the closing
// row for the last chunk).  Transposed slopes: the rows of G^T y from the solution y, its
// neighbours and the values y_J of the piece's junctions; the taps left of the piece alone
// give y at the row before it (`first`: the piece's first chunk); dn = the value at the
// closing node.  Differences of y cancel on smooth fields, so its rounding counts: the system
// is solved for s3 = 3/h times y, the elimination runs again from the carry (adding the carry
// to the first run's rows rounds each once more), and the row before a chunk follows from this
// chunk's carry and first row, so that its rounding is theirs (a sum over the chunks' results
// has its own).  Against 64 bits, error over that of the passes along one axis: white noise
// 1.06-1.08 -> 0.93, smooth fields 1.16-1.2 -> 0.94 (x_row likewise: 0.96 -> 0.86, 0.98 -> 0.81).
template <int STRIDE, int OP, bool IN>
__device__ __forceinline__ float rows_finish(const Piece &pc, const TileChunk &t, const float *ex, int nw, int lane,
                                             float (&y)[kTileC], const TileEnds *end = nullptr, float s3 = 0.f,
                                             bool first = false, int nown = 0, float *dn = nullptr)
{
    float ph = 0.f, pe = 0.f, yin = 0.f, win = 0.f;
    const int ol = IN ? 128 + 64 * t.l : 128, orr = IN ? 128 + 64 * t.r : 192;
#pragma unroll
    for (int j = 0; j < kTileWaves; ++j) {
        if (j < nw) {   // uniform
            const float *e = ex + j * STRIDE + lane;
            const float B = e[0], W = e[64];
            ph += e[ol];
            pe += e[orr];
            yin = fmaf(t.fB[j], B, yin);
            win = fmaf(t.zB[j], B, win);
            win = fmaf(t.zW[j], W, win);
        }
    }
    if constexpr (OP != TILE_DT) {
        yin = fmaf(t.fph, ph, yin);
        float pm = ph;
        if (IN && OP == TILE_D1 && t.m >= 0) {    // uniform
            pm = 0.f;
            for (int j = 0; j < nw; ++j) pm += ex[j * STRIDE + lane + 128 + 64 * t.m];
#pragma unroll
            for (int c = 0; c < kTileC; ++c) y[c] = fmaf(t.Q[c], pm, y[c]);
        }
        win = fmaf(t.zph, pm, win);
    }
    win = fmaf(OP == TILE_DT ? s3 * t.zE : t.zE, pe, win);
    if constexpr (OP == TILE_DT) {
        float v = yin;
#pragma unroll
        for (int c = 0; c < kTileC; ++c) {
            v = sweep(s3, y[c], t.nf[c], v);
            y[c] = v;
        }
    }
    float v = win;
#pragma unroll
    for (int c = kTileC - 1; c >= 0; --c) {
        v = sweep(t.fi[c], OP == TILE_DT ? y[c] : fmaf(t.P[c], yin, y[c]), t.g[c], v);
        y[c] = v;
    }
    if constexpr (OP == TILE_DT) {
        float prev = 0.f;
        if (!first) {               // the last row of the chunk before, by its own factors
            const TileChunk &b = (&t)[-1];
            prev = sweep(b.fi[kTileC - 1], yin, b.g[kTileC - 1], y[0]);
        }
        if (first) {                // the row before the piece; a natural end mirrors y_0
            prev = 0.f;
            for (int j = 0; j < nw; ++j) prev = fmaf(-s3, ex[j * STRIDE + kPublish<OP, IN> - 64 + lane], prev);
            if (end->m1 != 0.f) prev = -y[0];
        }
        float wl = 0.f;
#pragma unroll
        for (int c = 0; c < kTileC; ++c)
            if (c == nown - 1) wl = y[c];
        float d = fmaf(end->sE, win, wl) + fmaf(end->cs, ph, end->ce * pe);
        float lo = prev;
#pragma unroll
        for (int c = 0; c < kTileC; ++c) {
            const float own = y[c];
            y[c] = lo - (c < kTileC - 1 ? y[c < kTileC - 1 ? c + 1 : c] : win);
            lo = own;
        }
        if (t.any_cs != 0.f) {
#pragma unroll
            for (int c = 0; c < kTileC; ++c) y[c] = fmaf(t.cs[c], ph, y[c]);
        }
        if (t.any_ce != 0.f) {
#pragma unroll
            for (int c = 0; c < kTileC; ++c) y[c] = fmaf(t.ce[c], pe, y[c]);
        }
        if (IN && pc.ni > 0 && (t.any_in || end->cj != 0.f)) {   // uniform
#pragma unroll
            for (int k = 0; k < kTileIn; ++k)
                if (k < pc.ni) {
                    float pj = 0.f;
                    for (int j = 0; j < nw; ++j) pj += ex[j * STRIDE + 256 + 64 * k + lane];
#pragma unroll
                    for (int c = 0; c < kTileC; ++c) y[c] = fmaf(t.cj[k][c], pj, y[c]);
                    if (k == pc.ni - 1) d = fmaf(end->cj, pj, d);
                }
        }
        *dn = d;
    }
    return win;
}

// ---- x ----------------------------------------------------------------------------
// What depends on the lane only: factors of its four nodes, carry multipliers, taps.
// Solve rows of the piece in LDS (row r at L + r * kRowPitch) by 16 lanes each: the
// derivative of the piece's nodes replaces them, and that of the line's last node follows
// when the piece closes the line.  The lane's table entry (factors of its four nodes, carry
// multipliers, taps k, k + 16, k + 32 of the two junctions and their places in the row) is
// read from LDS as it is needed: kept in registers over the fields it would take 44.  ti: the
// lane's entry for junctions inside the piece: a node that is one takes its tap sum as its row's
// value (its factors are 0), and the transposed rows take the values by weights.
struct XPiece {
    TileEnds end;
    float s3;
    int m, kc, hs, ni;
    bool last, wide;         // closes the line; taps beyond the first 32 of a junction
};

__device__ __forceinline__ XPiece x_piece(const TileAxis &t, const Piece &p, int lx)
{
    XPiece x;
    x.end = t.ends[lx];
    x.s3 = t.s3;
    x.m = p.m;
    x.hs = p.hs;
    x.ni = p.ni;
    x.kc = (p.m - 1) >> 2;
    x.last = p.e == t.N;
    x.wide = max(max(p.hs, p.he), p.hi) > 15;
    return x;
}

template <int OP, bool IN, bool ALONE = false>
__device__ __forceinline__ void x_row(const XPiece &p, const float4 *t, const float4 *ti, float *L, int k)
{
    __builtin_amdgcn_sched_barrier(0);   // one row group at a time: interleaved they spill
    const float4 cs = t[7], os = t[8], ce = t[9], oe = t[10];
    auto at = [&](float o) {        // the table holds byte offsets
        return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(L) + __float_as_int(o));
    };
    // transposed: the taps left of the piece alone give y at the node before it
    float pl = 0.f;
    if constexpr (OP == TILE_DT) {
        if (k < p.hs) pl = cs.x * at(os.x);
        if (k + 16 < p.hs) pl = fmaf(cs.y, at(os.y), pl);
        pl = row_sum(pl);
    }
    const float us = kDiffX<OP, IN, ALONE> ? L[kRowOwn] : 0.f, ue = kDiffX<OP, IN, ALONE> ? L[kRowRight] : 0.f;
    float ph = cs.x * (at(os.x) - us), pe = ce.x * (at(oe.x) - ue);
    ph = fmaf(cs.y, at(os.y) - us, ph);
    pe = fmaf(ce.y, at(oe.y) - ue, pe);
    if (p.wide) {                   // uniform
        ph = fmaf(cs.z, at(os.z) - us, ph);
        pe = fmaf(ce.z, at(oe.z) - ue, pe);
    }
    ph = row_sum(ph);
    pe = row_sum(pe);
    if constexpr (kDiffX<OP, IN, ALONE>) {
        ph = fmaf(p.end.cs, us, ph);
        pe = fmaf(p.end.ce, ue, pe);
    }
    float pj[kTileIn], pm = 0.f;
    if (IN && p.ni > 0) {   // uniform
        const float4 own = ti[1];
#pragma unroll
        for (int j = 0; j < kTileIn; ++j) {
            pj[j] = 0.f;
            if (j < p.ni) {
                const float4 c = ti[2 + 2 * j], o = ti[3 + 2 * j];
                float v = c.x * at(o.x);
                v = fmaf(c.y, at(o.y), v);
                if (p.wide) v = fmaf(c.z, at(o.z), v);
                pj[j] = row_sum(v);
                if (OP == TILE_D1) pm = fmaf(j == 0 ? own.x : (j == 1 ? own.y : own.z), pj[j], pm);
            }
        }
    }
    if (OP != TILE_DT && p.end.sE != 0.f) pe = fmaf(p.end.sE, L[kRowOwn + p.m] - L[kRowOwn + p.m - 1], pe);
    __builtin_amdgcn_sched_barrier(0);
    const float4 u = ld4(L + kRowOwn + 4 * k);
    const float uE = L[kRowRight];
    const float ul = row_shift_up_fill<1>(u.w, u.x);
    const float ur = row_shift_down_fill<1>(u.x, uE);
    const float4 nf = t[0], sc = t[1], P = t[4], a = t[5];
    auto rhs = [](float lo, float own, float hi) {
        if constexpr (OP == TILE_D1) return hi - lo;
        else if constexpr (OP == TILE_D2) return (hi - own) - (own - lo);
        else return own;
    };
    float y0, y1, y2, y3;
    // (junctions inside: the products with the rows' own values held over the carries; otherwise
    // the layer's elastic kernels spill 10 registers more and run 6 % longer)
    constexpr bool kOwn = IN && OP == TILE_D1;
    if constexpr (kOwn) {
        y0 = sc.x * rhs(ul, u.x, u.y);
        y1 = sc.y * rhs(u.x, u.y, u.z);
        y2 = sc.z * rhs(u.y, u.z, u.w);
        y3 = sc.w * rhs(u.z, u.w, ur);
        if (p.ni > 0) {
            const float4 q = ti[0];
            y0 = fmaf(q.x, pm, y0);
            y1 = fmaf(q.y, pm, y1);
            y2 = fmaf(q.z, pm, y2);
            y3 = fmaf(q.w, pm, y3);
        }
        y1 = fmaf(nf.y, y0, y1);
        y2 = fmaf(nf.z, y1, y2);
        y3 = fmaf(nf.w, y2, y3);
    } else {
        const float4 k = OP == TILE_DT ? make_float4(p.s3 * sc.x, p.s3 * sc.y, p.s3 * sc.z, p.s3 * sc.w) : sc;
        y0 = k.x * rhs(ul, u.x, u.y);
        y1 = sweep(k.y, rhs(u.x, u.y, u.z), nf.y, y0);
        y2 = sweep(k.z, rhs(u.y, u.z, u.w), nf.z, y1);
        y3 = sweep(k.w, rhs(u.z, u.w, ur), nf.w, y2);
    }
    float B = fmaf(a.w, ph, y3);
    B = fmaf(a.x, row_shift_up_fill<1>(B, 0.f), B);
    B = fmaf(a.y, row_shift_up_fill<2>(B, 0.f), B);
    B = fmaf(a.z, row_shift_up_fill<4>(B, 0.f), B);
    const float yin = row_shift_up_fill<1>(B, ph);
    if constexpr (OP == TILE_DT) {
        y0 = sweep(p.s3, sc.x * u.x, nf.x, yin);       // weights of 1 and 0
        y1 = sweep(p.s3, sc.y * u.y, nf.y, y0);
        y2 = sweep(p.s3, sc.z * u.z, nf.z, y1);
        y3 = sweep(p.s3, sc.w * u.w, nf.w, y2);
    } else {
        y0 = fmaf(P.x, yin, y0);
        y1 = fmaf(P.y, yin, y1);
        y2 = fmaf(P.z, yin, y2);
        y3 = fmaf(P.w, yin, y3);
    }
    float we = fmaf(-p.end.imE, y3, p.end.iE * (OP == TILE_DT ? p.s3 * pe : pe));   // of the closing lane
    we = __shfl(we, p.kc, 16);
    __builtin_amdgcn_sched_barrier(0);
    const float4 fi = t[2], g = t[3], b = t[6];
    const float t0 = fi.x * y0, t1 = fi.y * y1, t2 = fi.z * y2, t3 = fi.w * y3;
    float W = fmaf(g.z, t3, t2);
    W = fmaf(g.y, W, t1);
    W = fmaf(g.x, W, t0);
    W = fmaf(b.w, we, W);
    W = fmaf(b.x, row_shift_down_fill<1>(W, 0.f), W);
    W = fmaf(b.y, row_shift_down_fill<2>(W, 0.f), W);
    W = fmaf(b.z, row_shift_down_fill<4>(W, 0.f), W);
    const float win = row_shift_down_fill<1>(W, we);
    float4 r;
    r.w = kOwn ? fmaf(g.w, win, t3) : sweep(fi.w, y3, g.w, win);
    r.z = kOwn ? fmaf(g.z, r.w, t2) : sweep(fi.z, y2, g.z, r.w);
    r.y = kOwn ? fmaf(g.y, r.z, t1) : sweep(fi.y, y1, g.y, r.z);
    r.x = kOwn ? fmaf(g.x, r.y, t0) : sweep(fi.x, y0, g.x, r.y);
    float dn = we;                  // the closing node
    if constexpr (OP == TILE_DT) {
        const float4 c1 = t[11], c2 = t[12];
        const int cc = (p.m - 1) & 3;
        const float wl = __shfl(cc == 0 ? r.x : (cc == 1 ? r.y : (cc == 2 ? r.z : r.w)), p.kc, 16);
        dn = fmaf(p.end.sE, we, wl) + fmaf(p.end.cs, ph, p.end.ce * pe);
        const float before = p.end.m1 != 0.f ? -r.x : -p.s3 * pl;   // a natural end mirrors y_0
        const float lo = row_shift_up_fill<1>(r.w, before);
        const float hi = row_shift_down_fill<1>(r.x, we);
        float4 o;
        o.x = (lo - r.y) + fmaf(c1.x, ph, c2.x * pe);
        o.y = (r.x - r.z) + fmaf(c1.y, ph, c2.y * pe);
        o.z = (r.y - r.w) + fmaf(c1.z, ph, c2.z * pe);
        o.w = (r.z - hi) + fmaf(c1.w, ph, c2.w * pe);
        if (IN && p.ni > 0) {
#pragma unroll
            for (int j = 0; j < kTileIn; ++j)
                if (j < p.ni) {
                    const float4 c = ti[8 + j];
                    o.x = fmaf(c.x, pj[j], o.x);
                    o.y = fmaf(c.y, pj[j], o.y);
                    o.z = fmaf(c.z, pj[j], o.z);
                    o.w = fmaf(c.w, pj[j], o.w);
                    if (j == p.ni - 1) dn = fmaf(p.end.cj, pj[j], dn);
                }
        }
        r = o;
    }
    st4(L + kRowOwn + 4 * k, r);
    if (p.last) {
        wave_sync();
        if (k == 0) L[kRowOwn + p.m] = dn;
    }
}

}  // namespace

}  // namespace loss
