// Single-axis passes (gfx950): one operator along one axis of a batch of fields, read from
// and written to the caller's arrays: the slopes and moments of loss_deriv (paper Sec. 3.1-
// 3.2, eq. derivative_approximation) and the transposed slopes of the adjoints.
//
// Transposed slopes D^T = G^T T^{-T}: a piece's interior system is closed (junction rows of
// T are identity rows); y at a junction is z_J minus the neighbouring interior values, which
// are sums over the pieces on either side with weights that decay by 0.27 per node, so they
// are taps like the slopes' own.  One kernel thus does what took three (interior solve,
// junction rows, gather): 16 bytes per node (in, coefficient, target) instead of 24.
//
// Bound by HBM; derivatives of user arrays spent half their time on copies into and out of
// padded rows, one field at a time.  Measured: order 2 along z of 2 x 257^3 254 -> 77 us a
// call; transposed along y of 3 x 302x204x175 323 -> 86; D^T along z of 64 x 1025^2
// (accumulating, with coefficient) 380 -> 231 us (4.65 TB/s of 16 bytes per node).
#include "tile_device.h"

namespace loss {

namespace {

template <int OP, bool IN, bool RUNS>
__global__ void __launch_bounds__(kTileWaves * 64, 8) k_axis_rows(AxisArgs a, int ncg, int nreal)
{
    constexpr int kEx = kPublish<OP, IN>;
    __shared__ float ex[kTileWaves * kEx];
    const int lin = RUNS ? xcd_order(kXcdChunk) : xcd_range();
    if (lin >= nreal) return;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int per = ncg * a.t.nsub;
    const int o = lin / per, rem = lin - o * per;
    const int lr = rem / ncg, cg = rem - lr * ncg;
    const int o1 = o / a.n1, o0 = o - o1 * a.n1;
    const int64_t fb = o1 * a.s1 + o0 * a.s0;
    const Piece p = piece_of(a.t, lr);
    const bool lastr = p.e == a.t.N;
    const unsigned rs4 = 4u * (unsigned)a.stride;
    const int64_t col = (int64_t)cg * 64 + lane;
    const unsigned xc = (unsigned)min(col, a.ncol - 1);
    const bool act = col < a.ncol && (a.pitch == 0 || (int)(xc % (unsigned)a.pitch) < a.nx);
    const unsigned vx = 4u * xc;
    const int q = p.s + w * kTileC;
    const int nown = min(max(p.e - q, 0), kTileC);
    const bool clos = nown > 0 && q + kTileC >= p.e;          // holds the row before the closing one
    const int nh = halo_count(p);
    const int *hn = a.t.halo_node + (size_t)lr * kTapW;
    const float4 *hc = a.t.halo_c + (size_t)lr * kTapW;
    const Buf in = buf(a.in + fb), out = buf(a.out + fb);
    const bool has_c = OP == TILE_DT && a.coef != nullptr;    // uniform
    const Buf cf = buf(has_c ? a.coef + o0 * a.m0 : a.in);
    auto get = [&](int r) {
        const float v = ld(in, (unsigned)r * rs4, vx);
        return has_c ? v * ld(cf, (unsigned)r * rs4, vx) : v;
    };
    float u[kTileC + 2], yh[kHaloPre], y[kTileC], old[kTileC];
    u[0] = u[kTileC + 1] = 0.f;
#pragma unroll
    for (int c = 0; c < kTileC + 2; ++c)
        if (OP != TILE_DT || (c > 0 && c <= kTileC)) u[c] = get(max(min(q - 1 + c, p.e), 0));
#pragma unroll
    for (int h = 0; h < kHaloPre; ++h) yh[h] = get(hn[w + h * a.nw]);
    float us = 0.f, ue = 0.f;
    if constexpr (OP != TILE_DT) {                            // the junctions' own values
        us = get(p.s);
        ue = get(hn[p.hl]);
        if (OP == TILE_D2 && w == 0) u[0] = u[1];             // the first row's one-sided difference
    }
    if (OP == TILE_DT && a.accumulate) {
#pragma unroll
        for (int c = 0; c < kTileC; ++c) old[c] = ld(out, (unsigned)min(q + c, p.e) * rs4, vx);
    }
    const TileChunk &rt = a.t.chunk[(size_t)lr * kTileWaves + w];
    const TileEnds end = a.t.ends[lr];
    float B, W;
    Taps tp;
    rows_local<OP>(rt, u, y, B, W, a.t.s3);
    taps_own<OP, IN>(rt, u, us, ue, tp);
#pragma unroll
    for (int h = 0; h < kHaloPre; ++h) taps_halo<OP, IN>(p, hc, w + h * a.nw, yh[h], us, ue, tp);
    for (int i = w + kHaloPre * a.nw; i < nh; i += a.nw) taps_halo<OP, IN>(p, hc, i, get(hn[i]), us, ue, tp);
    if (OP != TILE_DT && w == 0) {
        tp.s = fmaf(end.cs, us, tp.s);
        tp.e = fmaf(end.ce, ue, tp.e);
    }
    if (OP != TILE_DT && clos) {
        float u1 = 0.f, u0 = 0.f;
#pragma unroll
        for (int c = 0; c < kTileC; ++c)
            if (c == nown - 1) { u0 = u[c + 1]; u1 = u[c + 2]; }
        tp.e = fmaf(end.sE, u1 - u0, tp.e);
    }
    rows_publish<OP, IN>(p, ex + w * kEx, lane, B, W, tp);
    __syncthreads();
    if (nown == 0) return;
    float dn = 0.f;
    const float we = rows_finish<kEx, OP, IN>(p, rt, ex, a.nw, lane, y, &end, a.t.s3, w == 0, nown, &dn);
    if (OP != TILE_DT) dn = we;
    if (!act) return;
#pragma unroll
    for (int c = 0; c < kTileC; ++c)
        if (c < nown) {
            const unsigned r = (unsigned)(q + c) * rs4;
            st(out, r, vx, OP == TILE_DT && a.accumulate ? fmaf(a.alpha, y[c], old[c]) : y[c]);
        }
    if (clos && lastr) {
        const unsigned r = (unsigned)p.e * rs4;
        st(out, r, vx, OP == TILE_DT && a.accumulate ? fmaf(a.alpha, dn, ld(out, r, vx)) : dn);
    }
}

// Along x: a wave takes one piece of 8 lines (lane = node in and out, any alignment), the
// four waves of a workgroup the same piece of consecutive lines.
constexpr int kXWaves = 4;

template <int OP, bool IN>
__global__ void __launch_bounds__(kXWaves * 64) k_axis_x(AxisArgs a, int ngrp, int nreal)
{
    __shared__ float4 tab4[16 * (kLaneF / 4)], tabi4[IN ? 16 * (kLaneInF / 4) : 1];
    __shared__ float4 lds4[kXWaves * kWaveLds / 4];
    const int lin = xcd_range();
    if (lin >= nreal) return;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int grp = lin / a.t.nsub, lx = lin - grp * a.t.nsub;
    const Piece p = piece_of(a.t, lx);
    const int64_t line0 = ((int64_t)grp * kXWaves + w) * kTileC;
    const int nl = (int)max((int64_t)0, min((int64_t)kTileC, a.n_outer - line0));
    float *L = reinterpret_cast<float *>(lds4) + w * kWaveLds;
    const unsigned rs4 = 4u * (unsigned)a.s0;
    const int64_t lb = min(line0, a.n_outer - 1);             // waves past the last line repeat it
    const Buf in = buf(a.in + lb * a.s0), out = buf(a.out + lb * a.s0);
    const int nh = halo_count(p);
    const bool wide = nh > 32;
    const int hi = min(lane & 31, nh - 1), hj = min(32 + (lane & 15), nh - 1);
    const unsigned vx = 4u * (unsigned)min(p.s + lane, p.e);
    const unsigned hcol = 4u * line_node(halo_pos(p, hi), a.t.N, a.t.periodic);
    const unsigned wcol = 4u * line_node(halo_pos(p, hj), a.t.N, a.t.periodic);
    auto row = [&](int c) { return (unsigned)max(min(c, nl - 1), 0) * rs4; };
    float u[kTileC], xh[6];
#pragma unroll
    for (int c = 0; c < kTileC; ++c) u[c] = ld(in, row(c), vx);
#pragma unroll
    for (int h = 0; h < 4; ++h) xh[h] = ld(in, 0, row(2 * h + (lane >> 5)) + hcol);
    if (wide) {
#pragma unroll
        for (int h = 0; h < 2; ++h) xh[4 + h] = ld(in, 0, row(4 * h + (lane >> 4)) + wcol);
    }
    const float4 *tg = a.t.lanes + (size_t)lx * 16 * (kLaneF / 4);
    for (int i = threadIdx.x; i < 16 * (kLaneF / 4); i += kXWaves * 64) tab4[i] = tg[i];
    if (IN && p.ni > 0) {
        const float4 *ti = a.t.lanes_in + (size_t)lx * 16 * (kLaneInF / 4);
        for (int i = threadIdx.x; i < 16 * (kLaneInF / 4); i += kXWaves * 64) tabi4[i] = ti[i];
    }
    const XPiece xp = x_piece(a.t, p, lx);
#pragma unroll
    for (int c = 0; c < kTileC; ++c) L[c * kRowPitch + kRowOwn + lane] = u[c];
#pragma unroll
    for (int h = 0; h < 4; ++h) L[(2 * h + (lane >> 5)) * kRowPitch + halo_slot(p, hi)] = xh[h];
    if (wide) {
#pragma unroll
        for (int h = 0; h < 2; ++h) L[(4 * h + (lane >> 4)) * kRowPitch + halo_slot(p, hj)] = xh[4 + h];
    }
    __syncthreads();
    const int k = lane & 15;
#pragma unroll
    for (int it = 0; it < kTileC / 4; ++it)
        x_row<OP, IN, true>(xp, tab4 + k * (kLaneF / 4), tabi4 + k * (kLaneInF / 4), L + (4 * it + (lane >> 4)) * kRowPitch, k);
    wave_sync();
    if (lane >= p.m + (xp.last ? 1 : 0)) return;
#pragma unroll
    for (int c = 0; c < kTileC; ++c)
        if (c < nl) st(out, (unsigned)c * rs4, vx, L[c * kRowPitch + kRowOwn + lane]);
}

}  // namespace

hipError_t launch_axis_rows(int op, const AxisArgs &a, hipStream_t st)
{
    if (a.nw < 1 || a.nw > kTileWaves) return hipErrorInvalidValue;
    const int64_t ncg = (a.ncol + 63) / 64;
    const int64_t nreal = a.n_outer * ncg * a.t.nsub;
    if (nreal < 1 || nreal >= (1ll << 31) - 8) return hipErrorInvalidValue;
    const bool runs = ncg >= 64;   // see xcd_order
    const int64_t blocks = xcd_blocks(nreal, runs ? kXcdChunk : 1);
    if (blocks * 64 * a.nw >= 1ll << 32) return hipErrorInvalidValue;   // threads of a launch
    auto go = [&](auto k) { hipLaunchKernelGGL(k, (unsigned)blocks, 64 * a.nw, 0, st, a, (int)ncg, (int)nreal); };
    auto pick = [&](auto r) {
        constexpr bool R = decltype(r)::value;
        switch (op) {
        case TILE_D1: a.t.inside ? go(k_axis_rows<TILE_D1, true, R>) : go(k_axis_rows<TILE_D1, false, R>); return true;
        case TILE_D2: go(k_axis_rows<TILE_D2, false, R>); return true;
        case TILE_DT: a.t.inside ? go(k_axis_rows<TILE_DT, true, R>) : go(k_axis_rows<TILE_DT, false, R>); return true;
        }
        return false;
    };
    if (!(runs ? pick(std::true_type{}) : pick(std::false_type{}))) return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_axis_x(int op, const AxisArgs &a, hipStream_t st)
{
    const int64_t ngrp = (a.n_outer + kXWaves * kTileC - 1) / (kXWaves * kTileC);
    const int64_t nreal = ngrp * a.t.nsub;
    if (nreal < 1 || nreal >= (1ll << 31) - 8) return hipErrorInvalidValue;
    const unsigned blocks = (unsigned)((nreal + 7) / 8 * 8);
    if ((int64_t)blocks * kXWaves * 64 >= 1ll << 32) return hipErrorInvalidValue;   // threads of a launch
    auto go = [&](auto k) { hipLaunchKernelGGL(k, blocks, kXWaves * 64, 0, st, a, (int)ngrp, (int)nreal); };
    switch (op) {
    case TILE_D1: a.t.inside ? go(k_axis_x<TILE_D1, true>) : go(k_axis_x<TILE_D1, false>); break;
    case TILE_D2: go(k_axis_x<TILE_D2, false>); break;
    case TILE_DT: a.t.inside ? go(k_axis_x<TILE_DT, true>) : go(k_axis_x<TILE_DT, false>); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace loss
