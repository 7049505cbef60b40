// Tile passes (gfx950): the derivatives of a sub-flow along x and along one strided axis
// ("rows": y of an elastic grid, z of a 2-D acoustic one) in one kernel, combined with the
// update of the sub-flow's outputs (paper Sec. 2: the velocity-stress systems; Sec. 3.3:
// the Strang sub-flows), and the z derivatives an elastic stage needs beforehand.
//
// Why: the passes are bound by HBM.  One pass per derivative has to park the partial sums
// in full-size temporaries; taking two axes of a stage together leaves
//   acoustic, bytes per node and step: 60 (three line kernels) -> 44 (two tile kernels),
//   elastic: 264 (18 line kernels) -> 192 (two z stores of three fields, two tile kernels).
//
// A tile is a piece of at most 64 intervals of x times a piece of at most 64 intervals of
// the rows: patches longer than that are cut, and pieces of short patches reach across up to
// three junctions, whose slopes are tap sums like those of the ends and enter at their rows
// (8 x 1025^2 acoustic, patches of 16: 388 us per step with tiles of 16 x 16 nodes -> 105).
// A wave owns 8 consecutive rows, lane = column, so every row index, factor and carry
// coefficient along the rows is wave-uniform (scalar loads, SGPR operands) and every global
// access is one 256-byte row.
//
// The factors do not depend on the data, so neither do the multipliers of the carries:
//  * rows: each chunk of 8 rows eliminates and back-substitutes from zero carries and
//    publishes the two end values (B, W) and its share of the junction slopes' tap sums;
//    after ONE barrier every wave forms its two carries as sums over the chunks with
//    coefficients from the table (FP64 on the host), where composing the maps chunk by
//    chunk takes two barriers and the maps' multipliers through LDS.
//  * x: the wave's rows pass through LDS once (each wave its own rows, no barrier), 16 lanes
//    of four nodes solve a row, four rows at a time; the carries are composed by three
//    doubling steps of one DPP move and one FMA each.
// The tap sums along the rows come from the rows a wave holds and from the halo rows,
// which are dealt to the waves of the workgroup.
//
// Measured (us per step, line passes -> tiles): elastic 513^3 8150 -> 5860-6130, 257^3 x 2
// shots 2190 -> 1650, 65^3 155 -> 58; acoustic 2049^2 78 -> 62, 129^2 40 -> 21.  513^3: stress
// tiles 2400-2575 us (4.4-4.7 TB/s of the compulsory bytes), velocity tiles 1890-2019 (4.0-4.3),
// z stores 740-785 (4.1-4.4); a 1 GiB copy reaches 5.2 TB/s.
//
// What a tile does before its first field load counts: a per-tile word says whether it has
// receivers or a source (each tile walking the sources and the receivers' ranges, behind a
// read of the step counter: acoustic 2049^2 31.9 + 37.2 -> 28.4 + 32.0 us with the next).
//
// The adjoints' reverse steps run the same way with transposed slopes (TILE_*_T): x and row
// parts of D^T in one kernel, bytes per node and reverse step acoustic 68 -> 44, elastic
// 312 -> 216 and 20 launches fewer.  Measured (us per reverse step, without the gradient's
// sums): acoustic 64 x 1025^2 1165 -> 864, elastic 129^3 x 2 shots 540 -> 298.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "tile_device.h"

namespace loss {

namespace {

template <int MODE>
struct Traits;
struct Forward {
    static constexpr int OP = TILE_D1;
    static constexpr bool coef = false;           // inputs times c0
};
template <>
struct Traits<TILE_EL_STRESS> : Forward {   // v1 v2 v3
    static constexpr int SHAPE = TILE_EL_STRESS;  // which derivatives of which inputs, and their sums
    static constexpr int NF = 3;
    static constexpr bool xs(int f) { return true; }
    static constexpr bool ys(int f) { return true; }
    static constexpr int px(int f) { return 9 + 3 * f; }        // layer variable of d1 v_f, d2 v_f
    static constexpr int py(int f) { return 9 + 3 * f + 1; }
};
template <>
struct Traits<TILE_EL_VEL> : Forward {   // s11 s12 s22 s13 s23
    static constexpr int SHAPE = TILE_EL_VEL;
    static constexpr int NF = 5;
    static constexpr bool xs(int f) { return f == 0 || f == 1 || f == 3; }
    static constexpr bool ys(int f) { return f == 1 || f == 2 || f == 4; }
    static constexpr int px(int f) { return f == 0 ? 0 : (f == 1 ? 3 : 6); }
    static constexpr int py(int f) { return f == 1 ? 1 : (f == 2 ? 4 : 7); }
};
template <>
struct Traits<TILE_AC_STRESS> : Forward {   // v1 v3
    static constexpr int SHAPE = TILE_AC_STRESS;
    static constexpr int NF = 2;
    static constexpr bool xs(int f) { return f == 0; }
    static constexpr bool ys(int f) { return f == 1; }
    static constexpr int px(int f) { return 2; }
    static constexpr int py(int f) { return 3; }
};
template <>
struct Traits<TILE_AC_VEL> : Forward {   // sigma
    static constexpr int SHAPE = TILE_AC_VEL;
    static constexpr int NF = 1;
    static constexpr bool xs(int f) { return true; }
    static constexpr bool ys(int f) { return true; }
    static constexpr int px(int f) { return 0; }
    static constexpr int py(int f) { return 1; }
};

// Transposes: the transpose of a velocity pass takes the derivatives that the stress pass
// takes (sigma_ij bar += D_j^T (c0 u_i bar)) and the other way round.
template <>
struct Traits<TILE_EL_VEL_T> : Traits<TILE_EL_STRESS> {
    static constexpr int OP = TILE_DT;
    static constexpr bool coef = true;
};
template <>
struct Traits<TILE_EL_STRESS_T> : Traits<TILE_EL_VEL> {
    static constexpr int OP = TILE_DT;
};
template <>
struct Traits<TILE_AC_VEL_T> : Traits<TILE_AC_STRESS> {
    static constexpr int OP = TILE_DT;
    static constexpr bool coef = true;
};
template <>
struct Traits<TILE_AC_STRESS_T> : Traits<TILE_AC_VEL> {
    static constexpr int OP = TILE_DT;
    static constexpr bool coef = true;
};

template <int MODE>
constexpr int rows_slot(int f)
{
    int n = 0;
    for (int i = 0; i < f; ++i) n += Traits<MODE>::ys(i) ? 1 : 0;
    return n;
}

// floats of LDS of a wave: its rows of x, then what it publishes of each field
template <int MODE, bool IN>
constexpr int kModeLds = std::max(kWaveLds, rows_slot<MODE>(Traits<MODE>::NF) * kPublish<Traits<MODE>::OP, IN>);

// Sum of the source terms of field fid (a component of the outputs) over the R rows from
// row q on, as the update adds them.
template <int R>
__device__ __forceinline__ void source_add(const TileArgs &a, const Place &pl, int64_t n, int fid, int q,
                                           float (&add)[R])
{
#pragma unroll
    for (int c = 0; c < R; ++c) add[c] = 0.f;
    const int k1 = a.src_begin[pl.shot + 1];
    for (int k = a.src_begin[pl.shot]; k < k1; ++k) {
        const SrcDev &sd = a.src[k];
        if (fid < sd.field0 || fid >= sd.field0 + sd.nfield) continue;
        const int64_t ns = n + a.src_time_offset;
        if (ns < 0 || ns >= sd.nt) continue;
        const int r0 = a.row_axis == 1 ? sd.y0 : sd.z0, nr = a.row_axis == 1 ? sd.by : sd.bz;
        const int oo = a.row_axis == 1 ? pl.o - sd.z0 : 0, no = a.row_axis == 1 ? sd.bz : 1;
        if ((unsigned)oo >= (unsigned)no) continue;
        const float amp = a.src_scale * a.wavpool[sd.wav_off + ns];
        const unsigned ix = (unsigned)(pl.xc - sd.x0);
        const float *w = a.wpool + sd.w_off + (int64_t)oo * nr * sd.bx;
#pragma unroll
        for (int c = 0; c < R; ++c) {
            const unsigned ir = (unsigned)(q + c - r0);
            if (ir < (unsigned)nr && ix < (unsigned)sd.bx) {
                float v = amp * w[ir * (unsigned)sd.bx + ix];
                if (sd.force) v *= ld(buf(a.c0 + pl.mb), (unsigned)(q + c) * pl.rs4, pl.vx);
                add[c] += v;
            }
        }
    }
}

// The layer's sub-flow on one derivative of R rows: D becomes the effective derivative and
// the memory variable advances.  Along x the table entry is the lane's, along the rows the
// row's.  The memory values are requested before the solve whose result they meet (x: of
// the field, rows: before the barrier), and the rows' table entries before the first flow:
// one flow after the other, each waiting for its row's entry and value, was half of a tile's
// time in the layer (16 700 of 34 000 cycles, acoustic 1101 x 706).  184 x 142 x 211 with 16
// layer nodes: stress tiles 248 -> 192 us, velocity tiles 212 -> 170.  Kernels of their own:
// the values' registers and branches slowed those without a layer (z stores 204 -> 213 us).
template <int R>
__device__ __forceinline__ void layer_load(const TileArgs &a, const Place &pl, int var, int q, int last, bool on,
                                           float (&psi)[R])
{
    const Buf m = buf(a.pml_mem + var * a.pml_stride + pl.fb);
    if (!on) return;
#pragma unroll
    for (int c = 0; c < R; ++c) psi[c] = ld(m, (unsigned)min(q + c, last) * pl.rs4, pl.vx);
}

__device__ __forceinline__ bool layer_band(const TileAxis &ax, int j) { return j < ax.pml_w || j > ax.N - ax.pml_w; }

template <int R, bool ALONG_X>
__device__ __forceinline__ void layer_flow(const TileArgs &a, const Place &pl, int var, int q, int nrow, bool on,
                                           float4 tx, const float4 (&tr)[R], const float (&psi)[R], float (&D)[R])
{
    const Buf m = buf(a.pml_mem + var * a.pml_stride + pl.fb);
    if (!on) return;
#pragma unroll
    for (int c = 0; c < R; ++c)
        if (c < nrow && (ALONG_X || layer_band(a.r, q + c))) {
            float psi1;
            D[c] = pml_flow(ALONG_X ? tx : tr[c], D[c], psi[c], &psi1);
            if (a.pml_store) st(m, (unsigned)(q + c) * pl.rs4, pl.vx, psi1);
        }
}

// What the update of a row takes: the sums of x and row derivatives per output.
//   elastic stress: d1 v1, d2 v2, d2 v1 + d1 v2, d1 v3, d2 v3; elastic velocity:
//   d1 s_i1 + d2 s_i2; acoustic stress: d1 v1 + d3 v3; acoustic velocity: d1 sigma, d3 sigma
template <int SHAPE>
struct SumsOf;
template <>
struct SumsOf<TILE_EL_STRESS> { static constexpr int N = 5; };
template <>
struct SumsOf<TILE_EL_VEL> { static constexpr int N = 3; };
template <>
struct SumsOf<TILE_AC_STRESS> { static constexpr int N = 1; };
template <>
struct SumsOf<TILE_AC_VEL> { static constexpr int N = 2; };

template <int MODE>
using Sums = SumsOf<Traits<MODE>::SHAPE>;

template <int MODE, int R>
__device__ __forceinline__ void make_sums(const float (&dx)[Traits<MODE>::NF][R], const float (&dy)[Traits<MODE>::NF][R],
                                          float (&e)[Sums<MODE>::N][R])
{
    constexpr int SHAPE = Traits<MODE>::SHAPE;
#pragma unroll
    for (int c = 0; c < R; ++c) {
        if constexpr (SHAPE == TILE_EL_STRESS) {
            e[0][c] = dx[0][c];
            e[1][c] = dy[1][c];
            e[2][c] = dy[0][c] + dx[1][c];
            e[3][c] = dx[2][c];
            e[4][c] = dy[2][c];
        } else if constexpr (SHAPE == TILE_EL_VEL) {
            e[0][c] = dx[0][c] + dy[1][c];
            e[1][c] = dx[1][c] + dy[2][c];
            e[2][c] = dx[3][c] + dy[4][c];
        } else if constexpr (SHAPE == TILE_AC_STRESS) {
            e[0][c] = dy[1][c] + dx[0][c];
        } else {
            e[0][c] = dx[0][c];
            e[1][c] = dy[0][c];
        }
    }
}

// Update of the R rows from row q on, lane = column.  FULL: all R rows belong to the piece
// and no source reaches the tile (nearly all waves); else the first nrow rows, with the
// sources when srcs is set.  KEEP: the derivatives are stored too. 
template <int MODE, int R, bool FULL, bool KEEP>
__device__ __forceinline__ void tile_update(const TileArgs &a, const Place &pl, int64_t n, int q, int nrow, bool srcs,
                                            const float (&e)[Sums<MODE>::N][R])
{
    if (!pl.act) return;
    auto row = [&](int c) { return FULL || c < nrow; };
    auto get = [&](const float *p, int c) { return ld(buf(p + pl.fb), (unsigned)(q + c) * pl.rs4, pl.vx); };
    auto med = [&](const float *p, int c) { return ld(buf(p + pl.mb), (unsigned)(q + c) * pl.rs4, pl.vx); };
    auto put = [&](float *p, int c, float v) { st(buf(p + pl.fb), (unsigned)(q + c) * pl.rs4, pl.vx, v); };
    auto keep = [&](int k, int c, float v) {
        if (KEEP) put(a.keep + k * a.keep_stride, c, v);
    };
    float add[R];
#pragma unroll
    for (int c = 0; c < R; ++c) add[c] = 0.f;
    if constexpr (MODE == TILE_EL_STRESS) {
        if (!FULL && srcs) source_add<R>(a, pl, n, 3, q, add);   // stress sources act on the normal stresses alike
        constexpr int G = R < 4 ? R : 4;   // rows whose operands are in flight together
#pragma unroll
        for (int h = 0; h < R; h += G) {
            float s[3][G], t3[G], l2m[G], lam[G];
#pragma unroll
            for (int c = 0; c < G; ++c)
                if (row(h + c)) {
                    t3[c] = get(a.T[2], h + c);
                    l2m[c] = med(a.c0, h + c);
                    lam[c] = med(a.c1, h + c);
#pragma unroll
                    for (int i = 0; i < 3; ++i) s[i][c] = get(a.out[i], h + c);
                }
#pragma unroll
            for (int c = 0; c < G; ++c)
                if (row(h + c)) {
                    const float d[3] = {e[0][h + c], e[1][h + c], t3[c]};
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        const float other = i == 0 ? d[1] + d[2] : (i == 1 ? d[0] + d[2] : d[0] + d[1]);
                        float v = fmaf(l2m[c], d[i], lam[c] * other) + s[i][c];
                        if (!FULL) v += add[h + c];
                        put(a.out[i], h + c, v);
                        keep(i, h + c, d[i]);
                    }
                }
        }
#pragma unroll
        for (int h = 0; h < R; h += G) {
            float s[3][G], t1[G], t2[G], mu[G];
#pragma unroll
            for (int c = 0; c < G; ++c)
                if (row(h + c)) {
                    t1[c] = get(a.T[0], h + c);
                    t2[c] = get(a.T[1], h + c);
                    mu[c] = med(a.c2, h + c);
#pragma unroll
                    for (int i = 0; i < 3; ++i) s[i][c] = get(a.out[3 + i], h + c);
                }
#pragma unroll
            for (int c = 0; c < G; ++c)
                if (row(h + c)) {
                    const float gs[3] = {e[2][h + c], t1[c] + e[3][h + c], t2[c] + e[4][h + c]};
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        put(a.out[3 + i], h + c, fmaf(mu[c], gs[i], s[i][c]));
                        keep(3 + i, h + c, gs[i]);
                    }
                }
        }
    } else if constexpr (MODE == TILE_EL_VEL) {
        float b[R], v[3][R], t[3][R];
#pragma unroll
        for (int c = 0; c < R; ++c)
            if (row(c)) {
                b[c] = med(a.c0, c);
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    v[i][c] = get(a.base[i], c);
                    t[i][c] = get(a.T[i], c);
                }
            }
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            if (!FULL && srcs) source_add<R>(a, pl, n, i, q, add);
#pragma unroll
            for (int c = 0; c < R; ++c)
                if (row(c)) {
                    const float dr = e[i][c] + t[i][c];
                    float r = fmaf(a.alpha * b[c], dr, v[i][c]);
                    if (!FULL) r += add[c];
                    put(a.out[i], c, r);
                    keep(i, c, dr);
                }
        }
    } else if constexpr (MODE == TILE_AC_STRESS) {
        float s[R], K[R];
#pragma unroll
        for (int c = 0; c < R; ++c)
            if (row(c)) {
                s[c] = get(a.out[0], c);
                K[c] = med(a.c0, c);
            }
        if (!FULL && srcs) source_add<R>(a, pl, n, 0, q, add);
#pragma unroll
        for (int c = 0; c < R; ++c)
            if (row(c)) {
                float v = fmaf(a.alpha * K[c], e[0][c], s[c]);
                if (!FULL) v += add[c];
                put(a.out[0], c, v);
                keep(0, c, e[0][c]);
            }
    } else {
        float v1[R], v3[R], b[R], add3[R];
#pragma unroll
        for (int c = 0; c < R; ++c) {
            add3[c] = 0.f;
            if (row(c)) {
                b[c] = med(a.c0, c);
                v1[c] = get(a.base[0], c);
                v3[c] = get(a.base[1], c);
            }
        }
        if (!FULL && srcs) {
            source_add<R>(a, pl, n, 1, q, add);    // field ids of v1, v3
            source_add<R>(a, pl, n, 2, q, add3);
        }
#pragma unroll
        for (int c = 0; c < R; ++c)
            if (row(c)) {
                float p = fmaf(a.alpha * b[c], e[0][c], v1[c]), r = fmaf(a.alpha * b[c], e[1][c], v3[c]);
                if (!FULL) {
                    p += add[c];
                    r += add3[c];
                }
                put(a.out[0], c, p);
                put(a.out[1], c, r);
            }
    }
}

// The same for the transposes: the sums (and the stored z derivatives T) are added to the bars.
template <int MODE, int R, bool FULL>
__device__ __forceinline__ void tile_add(const TileArgs &a, const Place &pl, int q, int nrow,
                                         const float (&e)[Sums<MODE>::N][R])
{
    if (!pl.act) return;
    auto row = [&](int c) { return FULL || c < nrow; };
    auto get = [&](const float *p, int c) { return ld(buf(p + pl.fb), (unsigned)(q + c) * pl.rs4, pl.vx); };
    auto put = [&](float *p, int c, float v) { st(buf(p + pl.fb), (unsigned)(q + c) * pl.rs4, pl.vx, v); };
    // output j += sum of e[x] (if any) and T[t] (if any), R rows in flight
    auto add = [&](int j, int x, int t) {
        float o[R], z[R];
#pragma unroll
        for (int c = 0; c < R; ++c)
            if (row(c)) {
                o[c] = get(a.out[j], c);
                if (t >= 0) z[c] = get(a.T[t], c);
            }
#pragma unroll
        for (int c = 0; c < R; ++c)
            if (row(c)) {
                const float d = x < 0 ? z[c] : (t < 0 ? e[x < 0 ? 0 : x][c] : e[x < 0 ? 0 : x][c] + z[c]);
                put(a.out[j], c, fmaf(a.alpha, d, o[c]));
            }
    };
    if constexpr (MODE == TILE_EL_VEL_T) {
        add(0, 0, -1);
        add(1, 1, -1);
        add(2, -1, 2);
        add(3, 2, -1);
        add(4, 3, 0);
        add(5, 4, 1);
    } else if constexpr (MODE == TILE_EL_STRESS_T) {
        add(0, 0, 0);
        add(1, 1, 1);
        add(2, 2, 2);
    } else if constexpr (MODE == TILE_AC_VEL_T) {
        add(0, 0, -1);
    } else {
        add(0, 0, -1);
        add(1, 1, -1);
    }
}

// Waves per SIMD (registers): the elastic kernels hold three fields and their sums (121-123
// VGPRs: two workgroups per CU), the acoustic ones fit three (80 VGPRs).  Measured: acoustic
// 2049^2 29.4 + 37.2 us at two workgroups, 29.2 + 34.5 at three, 31.0 + 44.3 at four (spills);
// reading the updated arrays with the fields instead of after the solves 33.3 + 39.5.
template <int MODE>
constexpr int kTileWavesPerSimd = Traits<MODE>::SHAPE == TILE_AC_STRESS || Traits<MODE>::SHAPE == TILE_AC_VEL ? 6 : 4;

template <int MODE, bool KEEP, bool LAYER, bool IN>
__global__ void __launch_bounds__(kTileWaves * 64, kTileWavesPerSimd<MODE>) k_tile(TileArgs a, int nreal, int chunk)
{
    using T = Traits<MODE>;
    constexpr int NF = T::NF, OP = T::OP, kLds = kModeLds<MODE, IN>, kEx = kPublish<OP, IN>;
    __shared__ float4 tab4[16 * (kLaneF / 4)];                // x lanes' table of the piece
    __shared__ float4 tabi4[IN ? 16 * (kLaneInF / 4) : 1];    // the same, junctions inside
    __shared__ float4 lds4[kTileWaves * kLds / 4];
    float *lds = reinterpret_cast<float *>(lds4);
    // (one run is left to the shifts: the division is 1 % of a 2049^2 acoustic step)
    const int lin = NF < 3 ? xcd_range() : xcd_order(chunk);
    if (lin >= nreal) return;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int ntx = a.x.nsub, ntr = a.r.nsub;
    const int plane = lin / (ntx * ntr), tile = lin - plane * (ntx * ntr);
    const int lr = tile / ntx, lx = tile - lr * ntx;
    Place pl;
    pl.shot = plane / a.nother;
    pl.o = plane - pl.shot * a.nother;
    pl.mb = pl.o * a.ostride;
    pl.fb = pl.shot * a.shot_stride + pl.mb;
    const Piece px = piece_of(a.x, lx), pr = piece_of(a.r, lr);
    const bool lastx = px.e == a.x.N, lastr = pr.e == a.r.N;
    pl.xc = min(px.s + lane, px.e);
    pl.act = lane < px.m + (lastx ? 1 : 0);

    // receivers of the tile and whether a source reaches it; nearly all tiles have neither,
    // and only the others wait for the step counter
    int rec0 = 0, nrec = 0;
    bool hits = false;
    if (a.info) {
        const int2 ti = a.info[lin];
        rec0 = ti.x;
        nrec = ti.y >> 1;
        hits = a.src && (ti.y & 1);
    }
    int64_t n = 0;
    if (nrec > 0 || hits) n = *a.step_in + a.step_add;
    if (a.step_out && blockIdx.x == 0 && threadIdx.x == 0) *a.step_out = *a.step_in + a.step_add;
    if (n < 1 || n > a.trace_len) nrec = 0;
    if ((MODE == TILE_EL_VEL || MODE == TILE_AC_VEL) && nrec > 0) {   // half of the old value
        for (int k = rec0 + (int)threadIdx.x; k < rec0 + nrec; k += blockDim.x) {
            const RecDev rd = a.rec[k];
            a.traces[rd.trace_off + n - 1] = 0.5 * (double)a.fields[rd.comp][rd.shot * a.shot_stride + rd.node];
        }
        __syncthreads();
    }

    const int q = pr.s + w * kTileC;
    const int nown = min(max(pr.e - q, 0), kTileC);           // rows of the piece in this wave
    const bool clos = lastr && nown > 0 && q + kTileC >= pr.e;  // this wave also updates row N
    float *L = lds + w * kLds;
    pl.vx = 4u * pl.xc;
    pl.rs4 = 4u * (unsigned)a.rstride;

    // ---- loads ---------------------------------------------------------------------
    // the x table first: the barrier it needs then does not wait for the fields
    constexpr int kTab = 16 * (kLaneF / 4);
    const float4 *tabg = a.x.lanes + (size_t)lx * kTab;
    const float4 tab_reg = tabg[min((int)threadIdx.x, kTab - 1)];
    // rows past the piece repeat its closing row (their factors ignore them)
    float u[NF][kTileC + 2], yh[NF][kHaloPre], xh[NF][6];
    const int nhx = halo_count(px), nhr = halo_count(pr);
    const int *hn = a.r.halo_node + (size_t)lr * kTapW;
    const float4 *hc = a.r.halo_c + (size_t)lr * kTapW;
    // x halo: entries 0 .. 31 of two rows per load, entries 32 .. 40 (wide taps) of four
    const bool wide = nhx > 32;
    const int hi = min(lane & 31, nhx - 1), hj = min(32 + (lane & 15), nhx - 1);
    const unsigned hcol = 4u * line_node(halo_pos(px, hi), a.x.N, a.x.periodic);
    auto load = [&](int f) {
        const Buf in = buf(a.in[f] + pl.fb);
#pragma unroll
        for (int c = 0; c < kTileC + 2; ++c)
            if ((T::ys(f) && OP == TILE_D1) || (c > 0 && c <= kTileC))
                u[f][c] = ld(in, (unsigned)max(min(q - 1 + c, pr.e), 0) * pl.rs4, pl.vx);
        if (T::xs(f)) {
#pragma unroll
            for (int h = 0; h < 4; ++h)
                xh[f][h] = ld(in, 0, (unsigned)min(q + 2 * h + (lane >> 5), pr.e) * pl.rs4 + hcol);
            if (wide) {
                const unsigned wcol = 4u * line_node(halo_pos(px, hj), a.x.N, a.x.periodic);
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    xh[f][4 + h] = ld(in, 0, (unsigned)min(q + 4 * h + (lane >> 4), pr.e) * pl.rs4 + wcol);
            }
        }
    };
    const Buf cf = buf(T::coef ? a.c0 + pl.mb : a.in[0]);
    auto scale = [&](int f) {       // inputs times their coefficient
#pragma unroll
        for (int c = 1; c <= kTileC; ++c) u[f][c] *= ld(cf, (unsigned)max(min(q - 1 + c, pr.e), 0) * pl.rs4, pl.vx);
        if (T::xs(f)) {
#pragma unroll
            for (int h = 0; h < 4; ++h) xh[f][h] *= ld(cf, 0, (unsigned)min(q + 2 * h + (lane >> 5), pr.e) * pl.rs4 + hcol);
            if (wide) {
                const unsigned wcol = 4u * line_node(halo_pos(px, hj), a.x.N, a.x.periodic);
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    xh[f][4 + h] *= ld(cf, 0, (unsigned)min(q + 4 * h + (lane >> 4), pr.e) * pl.rs4 + wcol);
            }
        }
    };
    auto load_halo = [&](int f) {   // entries past the halo's count repeat row e with zero taps
#pragma unroll
        for (int h = 0; h < kHaloPre; ++h) {
            const unsigned r = (unsigned)hn[w + h * a.nw] * pl.rs4;
            yh[f][h] = ld(buf(a.in[f] + pl.fb), r, pl.vx);
            if (T::coef) yh[f][h] *= ld(cf, r, pl.vx);
        }
    };
#pragma unroll
    for (int f = 0; f < NF; ++f)
        if (T::xs(f)) load(f);
    if (T::coef) {
#pragma unroll
        for (int f = 0; f < NF; ++f)
            if (T::xs(f)) scale(f);
    }
    const TileChunk &rt = a.r.chunk[(size_t)lr * kTileWaves + w];
    const float rend = a.r.ends[lr].sE;
    const int k16 = lane & 15;
    const float4 *xt = tab4 + k16 * (kLaneF / 4);
    const float4 *xti = tabi4 + k16 * (kLaneInF / 4);
    const XPiece xp = x_piece(a.x, px, lx);
    if ((int)threadIdx.x < kTab) tab4[threadIdx.x] = tab_reg;
    for (int i = threadIdx.x + blockDim.x; i < kTab; i += blockDim.x) tab4[i] = tabg[i];   // fewer than four waves
    if (IN && px.ni > 0) {
        constexpr int kTabIn = 16 * (kLaneInF / 4);
        for (int i = threadIdx.x; i < kTabIn; i += blockDim.x) tabi4[i] = a.x.lanes_in[(size_t)lx * kTabIn + i];
    }
    __syncthreads();                                          // the lanes' table

    // ---- x: the wave's rows through LDS -------------------------------------------------
    const bool xband = LAYER && (px.s < a.x.pml_w || px.e > a.x.N - a.x.pml_w);   // uniform
    const bool xon = xband && pl.act && layer_band(a.x, pl.xc);
    float4 xt4{};
    if (xband) xt4 = a.px[pl.xc];
    float dx[NF][kTileC], dy[NF][kTileC], dxn[NF][1], dyn[NF][1];
    float *L16 = L + (lane >> 4) * kRowPitch;
    float *Lh = L + (lane >> 5) * kRowPitch + halo_slot(px, hi), *Lw = L + (lane >> 4) * kRowPitch + halo_slot(px, hj);
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        if (T::xs(f) && nown > 0) {
            float psi[kTileC];
            if (xband) layer_load<kTileC>(a, pl, T::px(f), q, pr.e, xon, psi);
            wave_sync();
#pragma unroll
            for (int c = 0; c < kTileC; ++c) L[c * kRowPitch + kRowOwn + lane] = u[f][c + 1];
#pragma unroll
            for (int h = 0; h < 4; ++h) Lh[2 * h * kRowPitch] = xh[f][h];
            if (wide) {
#pragma unroll
                for (int h = 0; h < 2; ++h) Lw[4 * h * kRowPitch] = xh[f][4 + h];
            }
            wave_sync();
#pragma unroll
            for (int it = 0; it < kTileC / 4; ++it) x_row<OP, IN>(xp, xt, xti, L16 + 4 * it * kRowPitch, k16);
            wave_sync();
#pragma unroll
            for (int c = 0; c < kTileC; ++c) dx[f][c] = L[c * kRowPitch + kRowOwn + lane];
            if (xband) layer_flow<kTileC, true>(a, pl, T::px(f), q, nown, xon, xt4, {}, psi, dx[f]);
            if (clos) {                   // row N of the line's last piece
                const Buf in = buf(a.in[f] + pl.fb);
                float un = ld(in, (unsigned)pr.e * pl.rs4, pl.vx);
                const int i = min(lane, nhx - 1);
                const unsigned xi = 4u * line_node(halo_pos(px, i), a.x.N, a.x.periodic);
                float xn = ld(in, (unsigned)pr.e * pl.rs4, xi);
                if (T::coef) {
                    un *= ld(cf, (unsigned)pr.e * pl.rs4, pl.vx);
                    xn *= ld(cf, (unsigned)pr.e * pl.rs4, xi);
                }
                wave_sync();
                L[kRowOwn + lane] = un;
                L[halo_slot(px, i)] = xn;
                wave_sync();
                x_row<OP, IN>(xp, xt, xti, L16, k16);
                wave_sync();
                dxn[f][0] = L[kRowOwn + lane];
                if (xband) {
                    float p1[1];
                    layer_load<1>(a, pl, T::px(f), pr.e, pr.e, xon, p1);
                    layer_flow<1, true>(a, pl, T::px(f), pr.e, 1, xon, xt4, {}, p1, dxn[f]);
                }
            }
        }
        if (f == 0) {                     // what the rows alone need, in flight during the x solves
#pragma unroll
            for (int g = 0; g < NF; ++g) {
                if (!T::xs(g)) {
                    load(g);
                    if (T::coef) scale(g);
                }
                if (T::ys(g)) load_halo(g);
            }
        }
    }

    // ---- rows: local elimination, shares of the tap sums ------------------------------
    wave_sync();
#pragma unroll
    for (int f = 0; f < NF; ++f)
        if (T::ys(f)) {
            float B, W;
            Taps tp;
            if (OP == TILE_DT) u[f][0] = u[f][kTileC + 1] = 0.f;
            rows_local<OP>(rt, u[f], dy[f], B, W, a.r.s3);
            taps_own<OP, IN>(rt, u[f], 0.f, 0.f, tp);
            // Right of the closing row the nearest come last; in the layer's kernels first: there
            // the other order costs registers (velocities of 16 x 1101 x 706 71 -> 79 us a kernel).
#pragma unroll
            for (int g = 0; g < kHaloPre; ++g) {
                const int h = LAYER ? g : kHaloPre - 1 - g;
                taps_halo<OP, IN>(pr, hc, w + h * a.nw, yh[f][h], 0.f, 0.f, tp);
            }
            for (int i = w + kHaloPre * a.nw; i < nhr; i += a.nw)     // few waves, wide taps
                taps_halo<OP, IN>(pr, hc, i,
                              ld(buf(a.in[f] + pl.fb), (unsigned)hn[i] * pl.rs4, pl.vx) *
                                  (T::coef ? ld(cf, (unsigned)hn[i] * pl.rs4, pl.vx) : 1.f),
                              0.f, 0.f, tp);
            if (OP == TILE_D1 && clos) {
                // natural end: the closing row's difference (rend is 0 on a junction)
                float ue = 0.f, ul = 0.f;
#pragma unroll
                for (int c = 0; c < kTileC; ++c)
                    if (c == nown - 1) { ul = u[f][c + 1]; ue = u[f][c + 2]; }
                tp.e = fmaf(rend, ue - ul, tp.e);
            }
            rows_publish<OP, IN>(pr, L + rows_slot<MODE>(f) * kEx, lane, B, W, tp);
        }
    // the layer: the wave's memory values of the rows
    const bool rband = LAYER && nown > 0 && (q < a.r.pml_w || min(q + kTileC, pr.e) > a.r.N - a.r.pml_w);   // uniform
    const bool ron = rband && pl.act;
    float psr[NF][kTileC];
    if (rband) {
#pragma unroll
        for (int f = 0; f < NF; ++f)
            if (T::ys(f)) layer_load<kTileC>(a, pl, T::py(f), q, pr.e, ron, psr[f]);
    }
    __syncthreads();
    if (nown > 0) {
#pragma unroll
        for (int f = 0; f < NF; ++f)
            if (T::ys(f)) {
                const float we = rows_finish<kLds, OP, IN>(pr, rt, lds + rows_slot<MODE>(f) * kEx, a.nw, lane, dy[f],
                                                       &a.r.ends[lr], a.r.s3, w == 0, nown, &dyn[f][0]);
                if (OP == TILE_D1) dyn[f][0] = we;
            }
        if (rband) {
            float4 t[kTileC], t1[1];
#pragma unroll
            for (int c = 0; c < kTileC; ++c) t[c] = a.pr[min(q + c, a.r.N)];
            t1[0] = a.pr[pr.e];
#pragma unroll
            for (int f = 0; f < NF; ++f)
                if (T::ys(f)) {
                    layer_flow<kTileC, false>(a, pl, T::py(f), q, nown, ron, {}, t, psr[f], dy[f]);
                    if (clos) {
                        float p1[1];
                        layer_load<1>(a, pl, T::py(f), pr.e, pr.e, ron, p1);
                        layer_flow<1, false>(a, pl, T::py(f), pr.e, 1, ron, {}, t1, p1, dyn[f]);
                    }
                }
        }
        float e[Sums<MODE>::N][kTileC], en[Sums<MODE>::N][1];
        make_sums<MODE, kTileC>(dx, dy, e);
        if constexpr (OP == TILE_DT) {
            if (nown == kTileC) tile_add<MODE, kTileC, true>(a, pl, q, kTileC, e);
            else tile_add<MODE, kTileC, false>(a, pl, q, nown, e);
        } else {
            if (!hits && nown == kTileC) tile_update<MODE, kTileC, true, KEEP>(a, pl, 0, q, kTileC, false, e);
            else tile_update<MODE, kTileC, false, KEEP>(a, pl, n, q, nown, hits, e);
        }
        if (clos) {
            make_sums<MODE, 1>(dxn, dyn, en);
            if constexpr (OP == TILE_DT) tile_add<MODE, 1, true>(a, pl, pr.e, 1, en);
            else tile_update<MODE, 1, false, KEEP>(a, pl, n, pr.e, 1, hits, en);
        }
    }
    if (nrec > 0) {   // uniform across the workgroup
        __syncthreads();
        for (int k = rec0 + (int)threadIdx.x; k < rec0 + nrec; k += blockDim.x) {
            const RecDev rd = a.rec[k];
            const double v = (double)a.fields[rd.comp][rd.shot * a.shot_stride + rd.node];
            double *t = a.traces + rd.trace_off + n - 1;
            if (MODE == TILE_EL_VEL || MODE == TILE_AC_VEL) *t += 0.5 * v;
            else *t = v;
        }
    }
}

// ---- z derivatives of an elastic stage ------------------------------------------------
// One workgroup per (field, shot, 64 flattened columns of an x-y plane, piece of z); the
// transposes of the adjoint likewise.  The pieces of kZGroup neighbouring column groups
// follow each other: the rows that a piece takes from its neighbours are in the XCD's L2
// then, and the groups' rows still make runs of 8 KiB.  Measured, groups of a whole plane ->
// of 32: 513^3 818 -> 770 us (4.2 TB/s), 184 x 142 x 211 with layers 59 -> 56, 257^3 x 2 and
// 65^3 the same; 4, 8 and 16 groups lie between on 257^3 (206, 206, 204 us; 32: 200).
constexpr int kZGroup = 32;

template <int OP, bool LAYER, bool IN>
__global__ void __launch_bounds__(kTileWaves * 64, 8) k_tile_z(TileZArgs a, int ncg, int nreal)
{
    constexpr int kEx = kPublish<OP, IN>;
    __shared__ float ex[kTileWaves * kEx];
    const int lin = xcd_order(kXcdChunk);
    if (a.step_inc && blockIdx.x == 0 && threadIdx.x == 0) *a.step_inc += 1;
    if (lin >= nreal) return;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int per = ncg * a.r.nsub;                 // workgroups of one field of one shot
    const int fs = lin / per, rem = lin - fs * per;
    const int grp = rem / (kZGroup * a.r.nsub), g0 = grp * kZGroup;
    const int gw = min(kZGroup, ncg - g0);          // the last group is narrower
    const int in_g = rem - g0 * a.r.nsub, lr = in_g / gw, cg = g0 + in_g - lr * gw;
    const int f = fs / a.S, shot = fs - f * a.S;
    const float *in = (f == 0 ? a.in[0] : (f == 1 ? a.in[1] : a.in[2])) + shot * a.shot_stride;
    float *out = (f == 0 ? a.out[0] : (f == 1 ? a.out[1] : a.out[2])) + shot * a.shot_stride;
    float *mem = !LAYER ? nullptr : f == 0 ? a.pml_mem[0] : (f == 1 ? a.pml_mem[1] : a.pml_mem[2]);
    const Piece p = piece_of(a.r, lr);
    const bool lastr = p.e == a.r.N;
    const unsigned rs4 = 4u * (unsigned)a.plane;
    // columns past the plane are clamped; columns of the row padding are solved and not stored
    const unsigned xc = (unsigned)min((int64_t)cg * 64 + lane, a.plane - 1);
    const bool act = (int64_t)cg * 64 + lane < a.plane && (int)(xc % (unsigned)a.pitch) < a.nx;
    const unsigned vx = 4u * xc;
    const int q = p.s + w * kTileC;
    const int nown = min(max(p.e - q, 0), kTileC);
    const bool clos = lastr && nown > 0 && q + kTileC >= p.e;
    const int nh = halo_count(p);
    const int *hn = a.r.halo_node + (size_t)lr * kTapW;
    const float4 *hc = a.r.halo_c + (size_t)lr * kTapW;
    const Buf bin = buf(in);
    const bool has_c = OP == TILE_DT && a.coef != nullptr;    // uniform
    const Buf cf = buf(has_c ? a.coef : in);
    auto get = [&](int r) {
        const float v = ld(bin, (unsigned)r * rs4, vx);
        return has_c ? v * ld(cf, (unsigned)r * rs4, vx) : v;
    };
    float u[kTileC + 2], yh[kHaloPre], y[kTileC];
#pragma unroll
    for (int c = 0; c < kTileC + 2; ++c) u[c] = get(max(min(q - 1 + c, p.e), 0));
#pragma unroll
    for (int h = 0; h < kHaloPre; ++h) yh[h] = get(hn[w + h * a.nw]);
    const TileChunk &rt = a.r.chunk[(size_t)lr * kTileWaves + w];
    float B, W;
    Taps tp;
    rows_local<OP>(rt, u, y, B, W, a.r.s3);
    taps_own<OP, IN>(rt, u, 0.f, 0.f, tp);
#pragma unroll
    for (int h = kHaloPre - 1; h >= 0; --h) taps_halo<OP, IN>(p, hc, w + h * a.nw, yh[h], 0.f, 0.f, tp);
    for (int i = w + kHaloPre * a.nw; i < nh; i += a.nw) taps_halo<OP, IN>(p, hc, i, get(hn[i]), 0.f, 0.f, tp);
    if (OP == TILE_D1 && clos) {
        float ue = 0.f, ul = 0.f;
#pragma unroll
        for (int c = 0; c < kTileC; ++c)
            if (c == nown - 1) { ul = u[c + 1]; ue = u[c + 2]; }
        tp.e = fmaf(a.r.ends[lr].sE, ue - ul, tp.e);
    }
    rows_publish<OP, IN>(p, ex + w * kEx, lane, B, W, tp);
    // the layer's memory values of the wave's rows, requested before the barrier
    const int pw = a.r.pml_w;
    const bool band = LAYER && nown > 0 && (q < pw || min(q + kTileC, p.e) > a.r.N - pw);   // uniform
    const Buf m = buf(band ? mem + shot * a.shot_stride : in);
    float psi[kTileC];
    if (band) {
#pragma unroll
        for (int c = 0; c < kTileC; ++c) psi[c] = ld(m, (unsigned)min(q + c, p.e) * rs4, vx);
    }
    __syncthreads();
    if (nown == 0) return;
    float dn = 0.f;
    float we = rows_finish<kEx, OP, IN>(p, rt, ex, a.nw, lane, y, &a.r.ends[lr], a.r.s3, w == 0, nown, &dn);
    if (OP == TILE_DT) we = dn;
    if (!act) return;
    const Buf bout = buf(out);
    if (band) {
        const int N = a.r.N;
        float4 t[kTileC];
#pragma unroll
        for (int c = 0; c < kTileC; ++c) t[c] = a.pr[min(q + c, N)];
#pragma unroll
        for (int c = 0; c < kTileC; ++c)
            if (c < nown && (q + c < pw || q + c > N - pw)) {
                float psi1;
                y[c] = pml_flow(t[c], y[c], psi[c], &psi1);
                if (a.pml_store) st(m, (unsigned)(q + c) * rs4, vx, psi1);
            }
        if (clos && pw > 0) {
            float psi1;
            we = pml_flow(a.pr[N], we, ld(m, (unsigned)N * rs4, vx), &psi1);
            if (a.pml_store) st(m, (unsigned)N * rs4, vx, psi1);
        }
    }
#pragma unroll
    for (int c = 0; c < kTileC; ++c)
        if (c < nown) st(bout, (unsigned)(q + c) * rs4, vx, y[c]);
    if (clos) st(bout, (unsigned)p.e * rs4, vx, we);
}

}  // namespace

hipError_t launch_tile(int mode, const TileArgs &a, hipStream_t st)
{
    if (a.nw < 1 || a.nw > kTileWaves) return hipErrorInvalidValue;
    const int64_t nreal = (int64_t)a.S * a.nother * a.x.nsub * a.r.nsub;
    if (nreal < 1 || nreal >= (1ll << 31) - 8) return hipErrorInvalidValue;
    const bool elastic = mode == TILE_EL_STRESS || mode == TILE_EL_VEL || mode == TILE_EL_VEL_T || mode == TILE_EL_STRESS_T;
    const int chunk = elastic && nreal < 4096 ? a.x.nsub * std::max(1, (kXcdChunk + a.x.nsub / 2) / a.x.nsub)
                                              : (int)((nreal + 7) / 8);
    const int64_t blocks = xcd_blocks(nreal, chunk);
    if (blocks * 64 * a.nw >= 1ll << 32) return hipErrorInvalidValue;   // threads of a launch
    const int threads = 64 * a.nw, nr = (int)nreal;
    auto go = [&](auto k) { hipLaunchKernelGGL(k, (unsigned)blocks, threads, 0, st, a, nr, chunk); };
    const bool keep = a.keep != nullptr, layer = a.pml_mem != nullptr;
    if (mode >= TILE_EL_VEL_T && (keep || layer)) return hipErrorInvalidValue;
    auto pick = [&](auto in) {
        constexpr bool IN = decltype(in)::value;
        switch (mode) {
        case TILE_EL_STRESS:
            if (layer) keep ? go(k_tile<TILE_EL_STRESS, true, true, IN>) : go(k_tile<TILE_EL_STRESS, false, true, IN>);
            else keep ? go(k_tile<TILE_EL_STRESS, true, false, IN>) : go(k_tile<TILE_EL_STRESS, false, false, IN>);
            return true;
        case TILE_EL_VEL:
            if (layer) keep ? go(k_tile<TILE_EL_VEL, true, true, IN>) : go(k_tile<TILE_EL_VEL, false, true, IN>);
            else keep ? go(k_tile<TILE_EL_VEL, true, false, IN>) : go(k_tile<TILE_EL_VEL, false, false, IN>);
            return true;
        case TILE_AC_STRESS:
            if (layer) keep ? go(k_tile<TILE_AC_STRESS, true, true, IN>) : go(k_tile<TILE_AC_STRESS, false, true, IN>);
            else keep ? go(k_tile<TILE_AC_STRESS, true, false, IN>) : go(k_tile<TILE_AC_STRESS, false, false, IN>);
            return true;
        case TILE_AC_VEL:
            layer ? go(k_tile<TILE_AC_VEL, false, true, IN>) : go(k_tile<TILE_AC_VEL, false, false, IN>);
            return true;
        case TILE_EL_VEL_T: go(k_tile<TILE_EL_VEL_T, false, false, IN>); return true;
        case TILE_EL_STRESS_T: go(k_tile<TILE_EL_STRESS_T, false, false, IN>); return true;
        case TILE_AC_VEL_T: go(k_tile<TILE_AC_VEL_T, false, false, IN>); return true;
        case TILE_AC_STRESS_T: go(k_tile<TILE_AC_STRESS_T, false, false, IN>); return true;
        }
        return false;
    };
    if (!(a.x.inside || a.r.inside ? pick(std::true_type{}) : pick(std::false_type{}))) return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_tile_z(int op, const TileZArgs &a, hipStream_t st)
{
    if (a.nw < 1 || a.nw > kTileWaves || a.nf < 1 || a.nf > 3) return hipErrorInvalidValue;
    const int64_t ncg = (a.plane + 63) / 64;
    const int64_t nreal = (int64_t)a.nf * a.S * ncg * a.r.nsub;
    if (nreal >= (1ll << 31) - 8) return hipErrorInvalidValue;
    const int64_t blocks = xcd_blocks(nreal, kXcdChunk);
    if (blocks * 64 * a.nw >= 1ll << 32) return hipErrorInvalidValue;   // threads of a launch
    auto go = [&](auto k) { hipLaunchKernelGGL(k, (unsigned)blocks, 64 * a.nw, 0, st, a, (int)ncg, (int)nreal); };
    const bool layer = a.pml_mem[0] != nullptr;
    if (!(op == TILE_D1 || (op == TILE_DT && !layer))) return hipErrorInvalidValue;
    if (a.r.inside)
        op == TILE_DT ? go(k_tile_z<TILE_DT, false, true>)
                      : (layer ? go(k_tile_z<TILE_D1, true, true>) : go(k_tile_z<TILE_D1, false, true>));
    else
        op == TILE_DT ? go(k_tile_z<TILE_DT, false, false>)
                      : (layer ? go(k_tile_z<TILE_D1, true, false>) : go(k_tile_z<TILE_D1, false, false>));
    return hipGetLastError();
}

}  // namespace loss
