// Host check of the tile passes' tables and index arithmetic (tile_index.h, build_tile in
// tables.cpp).  For one axis it enumerates every index the kernels form along it (rows,
// halo rows, LDS places of the x solve) against the buffers' sizes, and evaluates the two
// solves as the kernels do (chunks of rows with summed carries; 16 lanes of four nodes with
// doubling steps) in FP32 on a random line, against the patch systems solved in FP64.
// Usage: tile_check N M halo end_mode.  Prints "ok" and the two relative errors.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "loss_internal.h"
#include "tile_index.h"

using namespace loss;

static int fails = 0;
static void check(bool ok, const char *what, long v, long lo, long hi)
{
    if (!ok && fails++ == 0) std::printf("%s = %ld outside [%ld, %ld)\n", what, v, lo, hi);
}
static void in(const char *what, long v, long lo, long hi) { check(v >= lo && v < hi, what, v, lo, hi); }

int main(int argc, char **argv)
{
    if (argc != 5) return 2;
    const int N = atoi(argv[1]), M = atoi(argv[2]), halo = atoi(argv[3]), mode = atoi(argv[4]);
    const double h = 10.0;
    const int per = mode == 2;
    AxisHost ax;
    std::string err = build_axis(ax, N, h, M, halo, mode);
    if (!err.empty()) { std::printf("%s\n", err.c_str()); return 1; }
    std::vector<float> u(N + 1);
    srand(7);
    for (float &v : u) v = (float)(rand() / (double)RAND_MAX - 0.5);
    if (per) u[N] = u[0];
    // T w = G u in FP64 (junction rows from the taps)
    std::vector<double> rhs(N + 1), w(N + 1);
    for (int i = 0; i <= N; ++i) {
        if (ax.slot[i] >= 0) {
            rhs[i] = 0;
            for (int t = 0; t < 2 * halo + 1; ++t) {
                const int k = ax.tap_idx[(size_t)ax.slot[i] * (2 * halo + 1) + t];
                if (k >= 0) rhs[i] += ax.tap_c[(size_t)ax.slot[i] * (2 * halo + 1) + t] * u[k];
            }
        } else {
            rhs[i] = ax.c0[i] * u[i] + (i > 0 ? ax.cm[i] * u[i - 1] : 0) + (i < N ? ax.cp[i] * u[i + 1] : 0);
        }
    }
    for (int i = 0; i <= N; ++i) w[i] = rhs[i] - (i > 0 ? ax.m[i] * w[i - 1] : 0);
    for (int i = N; i >= 0; --i) w[i] = (w[i] - (i < N ? ax.sup[i] * w[i + 1] : 0)) * ax.invd[i];

    double errs[2];
    for (int along_x = 0; along_x < 2; ++along_x) {
        TileHost t;
        err = build_tile(ax, along_x != 0, t);
        if (!err.empty()) { std::printf("%s\n", err.c_str()); return 1; }
        in("max_m", t.max_m, 1, kTileM + 1);
        std::vector<float> d(N + 1, NAN);
        for (int l = 0; l < t.nsub; ++l) {
            const Piece p = make_piece(t.piece[4 * l], t.piece[4 * l + 1], t.piece[4 * l + 2], t.piece[4 * l + 3]);
            const bool last = p.e == N;
            in("hl", p.hl, 0, kTileHalo + 1);
            in("hr", p.hr, 0, kTileHalo + 1);
            in("m", p.m, 1, (along_x && last ? kTileM - 1 : kTileM) + 1);
            auto node = [&](int k) { const int n = line_node(k, N, per); in("node", n, 0, N + 1); return n; };
            const float *end = &t.ends[(size_t)l * 4];
            if (!along_x) {
                const int nw = (t.max_m + kTileC - 1) / kTileC;
                std::vector<float> B(nw), W(nw), y((size_t)nw * kTileC);
                float ps = 0, pe = 0;
                for (int i = 0; i < halo_count(p); ++i) {
                    const int k = t.halo_node[(size_t)l * kTapW + i];
                    check(k == node(halo_pos(p, i)), "halo node", k, 0, N + 1);
                    ps += t.halo_c[2 * ((size_t)l * kTapW + i)] * u[k];
                    pe += t.halo_c[2 * ((size_t)l * kTapW + i) + 1] * u[k];
                }
                for (int j = 0; j < nw; ++j) {
                    const int q = p.s + j * kTileC;
                    float uu[kTileC + 2];
                    for (int c = 0; c < kTileC + 2; ++c) {
                        const int r = std::max(std::min(q - 1 + c, p.e), 0);
                        in("row", r, 0, N + 1);
                        uu[c] = q < p.e ? u[r] : 0.f;
                    }
                    const TileChunk &rt = ((const TileChunk *)t.chunk.data())[(size_t)l * kTileWaves + j];
                    float v = 0;
                    for (int c = 0; c < kTileC; ++c) {
                        v = rt.nf[c] * v + rt.sc[c] * (uu[c + 2] - uu[c]);
                        y[j * kTileC + c] = v;
                        ps += rt.ts[c] * uu[c + 1];
                        pe += rt.te[c] * uu[c + 1];
                        if (q + c == p.e - 1) pe += end[2] * (uu[c + 2] - uu[c + 1]);
                    }
                    B[j] = v;
                    v = 0;
                    for (int c = kTileC - 1; c >= 0; --c) v = rt.g[c] * v + rt.fi[c] * y[j * kTileC + c];
                    W[j] = v;
                }
                for (int j = 0; j < nw && p.s + j * kTileC < p.e; ++j) {
                    const TileChunk &ch = ((const TileChunk *)t.chunk.data())[(size_t)l * kTileWaves + j];
                    float yin = ch.fph * ps, win = ch.zph * ps + ch.zE * pe;
                    for (int i = 0; i < nw; ++i) {
                        yin += ch.fB[i] * B[i];
                        win += ch.zB[i] * B[i] + ch.zW[i] * W[i];
                    }
                    const int q = p.s + j * kTileC;
                    if (last && q + kTileC >= p.e) d[N] = win;
                    float v = win;
                    for (int c = kTileC - 1; c >= 0; --c) {
                        v = ch.g[c] * v + ch.fi[c] * (y[j * kTileC + c] + ch.P[c] * yin);
                        if (q + c < p.e) d[q + c] = v;
                    }
                }
            } else {
                std::vector<float> L(kRowPitch, NAN);
                for (int k = 0; k < kTileM; ++k) L[kRowOwn + k] = k <= p.m ? u[std::min(p.s + k, p.e)] : 0.f;
                for (int i = 0; i < halo_count(p); ++i) {
                    in("halo slot", halo_slot(p, i), 0, kRowPitch);
                    in("halo lane", i, 0, 64);
                    L[halo_slot(p, i)] = u[node(halo_pos(p, i))];
                }
                float ph = 0, pe = 0;
                const float *tab = &t.lanes[(size_t)l * 16 * kLaneF];
                for (int k = 0; k < 16; ++k)
                    for (int i = 0; i < 3; ++i) {
                        const float *x = tab + k * kLaneF;
                        int os, oe;
                        memcpy(&os, x + 32 + i, 4);
                        memcpy(&oe, x + 40 + i, 4);
                        in("tap place", os, 0, 4 * kRowPitch);
                        in("tap place", oe, 0, 4 * kRowPitch);
                        if (x[28 + i] != 0.f) ph += x[28 + i] * L[os / 4];
                        if (x[36 + i] != 0.f) pe += x[36 + i] * L[oe / 4];
                    }
                if (last) pe += end[2] * (L[kRowOwn + p.m] - L[kRowOwn + p.m - 1]);
                const int kc = (p.m - 1) / 4;
                float y[16][4], B[16], W[16], tt[16][4];
                for (int k = 0; k < 16; ++k) {
                    const float *x = tab + k * kLaneF;
                    float v = 0;
                    for (int c = 0; c < 4; ++c) {
                        const int i = 4 * k + c;
                        const float lo = i > 0 ? L[kRowOwn + i - 1] : L[kRowOwn], hi = i < 63 ? L[kRowOwn + i + 1] : L[kRowRight];
                        v = x[c] * v + x[4 + c] * (hi - lo);
                        y[k][c] = v;
                    }
                    B[k] = v + x[23] * ph;
                }
                auto scan = [&](float *v, int off, int dir) {
                    for (int s = 0; s < 3; ++s) {
                        float o[16];
                        for (int k = 0; k < 16; ++k) o[k] = v[k];
                        for (int k = 0; k < 16; ++k) {
                            const int j = k - dir * (1 << s);
                            v[k] = o[k] + tab[k * kLaneF + off + s] * (j >= 0 && j < 16 ? o[j] : 0.f);
                        }
                    }
                };
                scan(B, 20, 1);
                for (int k = 0; k < 16; ++k)
                    for (int c = 0; c < 4; ++c) y[k][c] += tab[k * kLaneF + 16 + c] * (k > 0 ? B[k - 1] : ph);
                const float we = end[0] * pe - end[1] * y[kc][3];
                for (int k = 0; k < 16; ++k) {
                    const float *x = tab + k * kLaneF;
                    float v = 0;
                    for (int c = 3; c >= 0; --c) { tt[k][c] = x[8 + c] * y[k][c]; v = x[12 + c] * v + tt[k][c]; }
                    W[k] = v + x[27] * we;
                }
                scan(W, 24, -1);
                for (int k = 0; k < 16; ++k) {
                    float v = k < 15 ? W[k + 1] : we;
                    for (int c = 3; c >= 0; --c) {
                        v = tab[k * kLaneF + 12 + c] * v + tt[k][c];
                        if (4 * k + c < p.m) d[p.s + 4 * k + c] = v;
                    }
                }
                if (last) d[N] = we;
            }
        }
        double a = 0, b = 0;
        for (int i = 0; i <= N; ++i) { a += (d[i] - w[i]) * (d[i] - w[i]); b += w[i] * w[i]; }
        errs[along_x] = std::sqrt(a / b);
    }
    if (fails) return 1;
    std::printf("ok %.2e %.2e\n", errs[0], errs[1]);
    return 0;
}
