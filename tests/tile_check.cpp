// Host check of the tile passes' tables and index arithmetic (tile_index.h, build_tile in
// tables.cpp).  For one axis and operator (0 slopes, 1 moments, 2 the transposed slopes) it
// enumerates every index the kernels form along it (rows, halo rows, LDS places of the x
// solve) against the buffers' sizes, and evaluates the two solves as the kernels do (chunks
// of rows with summed carries; 16 lanes of four nodes with doubling steps) in FP32 on a
// random line, against the patch systems solved in FP64.
// Usage: tile_check N M halo end_mode op across.  Prints "ok" and the two relative errors, or
// "unsupported" where build_tile refuses the transposed operator.
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

typedef std::vector<double> V;

// slopes of a line: T w = G u, junction rows from the taps
static V slopes(const AxisHost &ax, const V &u)
{
    const int N = ax.N, nt = 2 * ax.halo + 1;
    V w(N + 1);
    for (int i = 0; i <= N; ++i) {
        double r = 0;
        if (ax.slot[i] >= 0) {
            for (int t = 0; t < nt; ++t) {
                const int k = ax.tap_idx[(size_t)ax.slot[i] * nt + t];
                if (k >= 0) r += ax.tap_c[(size_t)ax.slot[i] * nt + t] * u[k];
            }
        } else {
            r = ax.c0[i] * u[i] + (i > 0 ? ax.cm[i] * u[i - 1] : 0) + (i < N ? ax.cp[i] * u[i + 1] : 0);
        }
        w[i] = r - (i > 0 ? ax.m[i] * w[i - 1] : 0);
    }
    for (int i = N; i >= 0; --i) w[i] = (w[i] - (i < N ? ax.sup[i] * w[i + 1] : 0)) * ax.invd[i];
    return w;
}

// moments, patch by patch
static V moments(const AxisHost &ax, const V &u)
{
    const int N = ax.N;
    const double h = ax.h;
    const V phi = slopes(ax, u);
    V out(N + 1, 0.0);
    for (int l = 0; l < ax.p; ++l) {
        const int s = l * ax.M, e = std::min(s + ax.M, N), n = e - s + 1;
        V a(n, 1.0), d(n, 4.0), c(n, 1.0), r(n);
        for (int i = 1; i < n - 1; ++i) r[i] = 6.0 / (h * h) * (u[s + i - 1] - 2 * u[s + i] + u[s + i + 1]);
        if (ax.kind[s] == ROW_NATURAL_L) { d[0] = 1; c[0] = 0; r[0] = 0; }
        else { d[0] = 2; r[0] = 6.0 / h * ((u[s + 1] - u[s]) / h - phi[s]); }
        if (ax.kind[e] == ROW_NATURAL_R) { d[n - 1] = 1; a[n - 1] = 0; r[n - 1] = 0; }
        else { d[n - 1] = 2; r[n - 1] = 6.0 / h * (phi[e] - (u[e] - u[e - 1]) / h); }
        for (int i = 1; i < n; ++i) { const double m = a[i] / d[i - 1]; d[i] -= m * c[i - 1]; r[i] -= m * r[i - 1]; }
        for (int i = n - 1; i >= 0; --i) {
            r[i] = (r[i] - (i + 1 < n ? c[i] * r[i + 1] : 0)) / d[i];
            if (i < n - 1 || e == N) out[s + i] = r[i];
        }
    }
    return out;
}

int main(int argc, char **argv)
{
    if (argc != 7) return 2;
    const int N = atoi(argv[1]), M = atoi(argv[2]), halo = atoi(argv[3]), mode = atoi(argv[4]), op = atoi(argv[5]), across = atoi(argv[6]);
    const double h = 10.0;
    const int per = mode == 2;
    AxisHost ax;
    std::string err = build_axis(ax, N, h, M, halo, mode);
    if (!err.empty()) { std::printf("%s\n", err.c_str()); return 1; }
    std::vector<float> u(N + 1);
    srand(7);
    for (float &v : u) v = (float)(rand() / (double)RAND_MAX - 0.5);
    if (per) u[N] = u[0];
    V ref(N + 1, 0.0);
    const V ud(u.begin(), u.end());
    if (op == 0) ref = slopes(ax, ud);
    else if (op == 1) ref = moments(ax, ud);
    else
        for (int j = 0; j <= N; ++j) {
            V unit(N + 1, 0.0);
            unit[j] = 1.0;
            const V col = slopes(ax, unit);
            for (int i = 0; i <= N; ++i) ref[j] += col[i] * ud[i];
        }
    const float s3 = (float)(3.0 / h);
    double errs[2];
    for (int along_x = 0; along_x < 2; ++along_x) {
        TileHost t;
        err = build_tile(ax, along_x != 0, op, across != 0, t);
        if (!err.empty()) { std::printf(op == 2 || across ? "unsupported %s\n" : "%s\n", err.c_str()); return op == 2 || across ? 0 : 1; }
        in("max_m", t.max_m, 1, kTileM + 1);
        std::vector<float> d(N + 1, NAN);
        for (int l = 0; l < t.nsub; ++l) {
            const Piece p = make_piece(t.piece[4 * l], t.piece[4 * l + 1], t.piece[4 * l + 2], t.piece[4 * l + 3]);
            check(p.s == t.sb[l] && p.e == t.sb[l + 1], "piece", p.s, 0, N);
            const bool last = p.e == N;
            in("hl", p.hl, 0, kTileHalo + 1);
            in("hr", p.hr, 0, kTileHalo + 1);
            in("ni", p.ni, 0, kTileIn + 1);
            if (op == 1 || !across) in("ni", p.ni, 0, 1);
            in("halo entries", halo_count(p), 1, kTapW + 1);
            in("m", p.m, 1, (along_x && last ? kTileM - 1 : kTileM) + 1);
            auto node = [&](int k) { const int n = line_node(k, N, per); in("node", n, 0, N + 1); return n; };
            TileEnds end;
            std::memcpy(&end, &t.ends[(size_t)l * 8], sizeof(end));
            const float us = op == 1 ? u[p.s] : 0.f, ue = op == 1 ? u[node(p.e)] : 0.f;   // moments: taps on differences
            float ps = op == 1 ? end.cs * us : 0.f, pe = op == 1 ? end.ce * ue : 0.f, pl = 0.f, pj[kTileIn] = {};
            if (!along_x) {
                const int nw = (t.max_m + kTileC - 1) / kTileC;
                const TileChunk *ch = (const TileChunk *)t.chunk.data() + (size_t)l * kTileWaves;
                std::vector<float> B(nw), W(nw), y((size_t)nw * kTileC), z((size_t)nw * kTileC);
                for (int i = 0; i < kTapW; ++i) {
                    const int k = t.halo_node[(size_t)l * kTapW + i];
                    in("halo node", k, 0, N + 1);
                    if (i < halo_count(p)) check(k == node(halo_pos(p, i)), "halo node", k, 0, N + 1);
                    const float *hc = &t.halo_c[4 * ((size_t)l * kTapW + i)];
                    ps += hc[0] * (u[k] - us);
                    if (i < p.hl) pl += hc[0] * u[k];
                    pe += hc[1] * (u[k] - ue);
                    if (p.ni > 0) pj[0] += hc[2] * u[k];
                    if (p.ni > 1) pj[p.ni - 1] += hc[3] * u[k];
                    else check(hc[3] == 0.f && (p.ni > 0 || hc[2] == 0.f), "halo tap", i, 0, 0);
                }
                for (int j = 0; j < nw; ++j) {
                    const int q = p.s + j * kTileC;
                    float uu[kTileC + 2];
                    for (int c = 0; c < kTileC + 2; ++c) {
                        const int r = std::max(std::min(q - 1 + c, p.e), 0);
                        in("row", r, 0, N + 1);
                        uu[c] = u[r];
                    }
                    if (op == 1 && j == 0) uu[0] = uu[1];
                    float v = 0;
                    for (int c = 0; c < kTileC; ++c) {
                        const float r = op == 0 ? uu[c + 2] - uu[c]
                                                : (op == 1 ? (uu[c + 2] - uu[c + 1]) - (uu[c + 1] - uu[c]) : uu[c + 1]);
                        v = ch[j].nf[c] * v + ch[j].sc[c] * r;
                        y[j * kTileC + c] = v;
                        ps += ch[j].ts[c] * (uu[c + 1] - us);
                        pe += ch[j].te[c] * (uu[c + 1] - ue);
                        for (int i = 0; i < kTileIn; ++i) {
                            pj[i] += ch[j].tj[i][c] * uu[c + 1];
                            check((i < p.ni && ch[j].any_in) || (ch[j].tj[i][c] == 0.f && ch[j].cj[i][c] == 0.f), "inside tap", i, 0, 0);
                        }
                        if (op != 2 && q + c == p.e - 1) pe += end.sE * (uu[c + 2] - uu[c + 1]);
                    }
                    B[j] = v;
                    v = 0;
                    for (int c = kTileC - 1; c >= 0; --c) v = ch[j].g[c] * v + ch[j].fi[c] * y[j * kTileC + c];
                    W[j] = v;
                }
                for (int j = 0; j < nw && p.s + j * kTileC < p.e; ++j) {
                    in("junction", ch[j].l, 0, 2 + p.ni);
                    in("junction", ch[j].r, 0, 2 + p.ni);
                    in("junction", ch[j].m, -1, 2 + p.ni);
                    auto jv = [&](int i) { return i == 0 ? ps : (i == 1 ? pe : pj[i - 2]); };
                    const float vl = jv(ch[j].l), vm = ch[j].m >= 0 ? jv(ch[j].m) : vl, vr = jv(ch[j].r);
                    float yin = ch[j].fph * vl, win = ch[j].zph * vm + ch[j].zE * vr, prev = ch[j].pE * pe;
                    for (int i = 0; i < nw; ++i) {
                        yin += ch[j].fB[i] * B[i];
                        win += ch[j].zB[i] * B[i] + ch[j].zW[i] * W[i];
                        prev += ch[j].pB[i] * B[i] + ch[j].pW[i] * W[i];
                    }
                    const int q = p.s + j * kTileC;
                    float v = win, w[kTileC];
                    for (int c = kTileC - 1; c >= 0; --c) {
                        v = ch[j].g[c] * v + ch[j].fi[c] * (y[j * kTileC + c] + (ch[j].m >= 0 ? ch[j].Q[c] * vm : 0.f) + ch[j].P[c] * yin);
                        w[c] = v;
                    }
                    if (op < 2) {
                        if (last && q + kTileC >= p.e) d[N] = win;
                        for (int c = 0; c < kTileC && q + c < p.e; ++c) d[q + c] = w[c];
                    } else {
                        if (j == 0) prev = end.m1 != 0.f ? -w[0] : -pl;
                        for (int c = 0; c < kTileC && q + c < p.e; ++c) {
                            const float lo = c > 0 ? w[c - 1] : prev, hi = c < kTileC - 1 ? w[c + 1] : win;
                            d[q + c] = s3 * (lo - hi) + ch[j].cs[c] * ps + ch[j].ce[c] * pe;
                            for (int i = 0; i < p.ni; ++i) d[q + c] += ch[j].cj[i][c] * pj[i];
                        }
                        if (last && q + kTileC >= p.e)
                            d[N] = s3 * (w[p.e - 1 - q] + end.sE * win) + end.cs * ps + end.ce * pe +
                                   (p.ni > 0 ? end.cj * pj[p.ni - 1] : 0.f);
                    }
                }
            } else {
                std::vector<float> L(kRowPitch, NAN);
                for (int k = 0; k < kTileM; ++k) L[kRowOwn + k] = u[std::min(p.s + k, p.e)];
                for (int i = 0; i < halo_count(p); ++i) {
                    in("halo slot", halo_slot(p, i), 0, kRowPitch);
                    in("halo lane", i, 0, 64);
                    L[halo_slot(p, i)] = u[node(halo_pos(p, i))];
                }
                const float *tab = &t.lanes[(size_t)l * 16 * kLaneF];
                for (int k = 0; k < 16; ++k)
                    for (int i = 0; i < 3; ++i) {
                        const float *x = tab + k * kLaneF;
                        int os, oe;
                        memcpy(&os, x + 32 + i, 4);
                        memcpy(&oe, x + 40 + i, 4);
                        in("tap place", os, 0, 4 * kRowPitch);
                        in("tap place", oe, 0, 4 * kRowPitch);
                        if (x[28 + i] != 0.f) ps += x[28 + i] * (L[os / 4] - us);
                        if (x[28 + i] != 0.f && k + 16 * i < p.hs) pl += x[28 + i] * L[os / 4];
                        if (x[36 + i] != 0.f) pe += x[36 + i] * (L[oe / 4] - ue);
                    }
                const float *tin = &t.lanes_in[(size_t)l * 16 * kLaneInF];
                for (int k = 0; k < 16; ++k)
                    for (int j = 0; j < kTileIn; ++j)
                        for (int i = 0; i < 3; ++i) {
                            const float *x = tin + k * kLaneInF + 8 + 8 * j;
                            int o;
                            memcpy(&o, x + 4 + i, 4);
                            in("tap place", o, 0, 4 * kRowPitch);
                            check(j < p.ni || x[i] == 0.f, "inside tap", j, 0, 0);
                            check(i < 2 || std::max(std::max(p.hs, p.he), p.hi) > 15 || x[i] == 0.f, "third tap", j, 0, 0);
                            if (x[i] != 0.f) pj[j] += x[i] * L[o / 4];
                        }
                if (op != 2) pe += end.sE * (u[p.e] - u[p.e - 1]);
                const int kc = (p.m - 1) / 4;
                float y[16][4], B[16], W[16], tt[16][4], w[65];
                for (int k = 0; k < 16; ++k) {
                    const float *x = tab + k * kLaneF;
                    float v = 0;
                    for (int c = 0; c < 4; ++c) {
                        const int i = 4 * k + c;
                        const float own = L[kRowOwn + i];
                        const float lo = i > 0 ? L[kRowOwn + i - 1] : own, hi = i < 63 ? L[kRowOwn + i + 1] : L[kRowRight];
                        const float *xi = tin + k * kLaneInF;
                        float pm = 0;
                        for (int j = 0; j < kTileIn; ++j) pm += xi[4 + j] * pj[j];
                        v = x[c] * v + xi[c] * pm + x[4 + c] * (op == 0 ? hi - lo : (op == 1 ? (hi - own) - (own - lo) : own));
                        y[k][c] = v;
                    }
                    B[k] = v + x[23] * ps;
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
                if (op == 2)
                    for (int k = 0; k < 1; ++k) B[0] = y[0][3];
                scan(B, 20, 1);
                for (int k = 0; k < 16; ++k)
                    for (int c = 0; c < 4; ++c) y[k][c] += tab[k * kLaneF + 16 + c] * (k > 0 ? B[k - 1] : (op == 2 ? 0.f : ps));
                const float we = end.iE * pe - end.imE * y[kc][3];
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
                        w[4 * k + c] = v;
                    }
                }
                w[64] = we;
                if (op < 2) {
                    for (int i = 0; i < p.m; ++i) d[p.s + i] = w[i];
                    if (last) d[N] = we;
                } else {
                    // past the closing lane the positions repeat the closing value
                    const float prev = end.m1 != 0.f ? -w[0] : -pl;
                    for (int i = 0; i < p.m; ++i) {
                        const float *x = tab + (i / 4) * kLaneF;
                        d[p.s + i] = s3 * ((i > 0 ? w[i - 1] : prev) - w[i + 1]) + x[44 + i % 4] * ps + x[48 + i % 4] * pe;
                        for (int j = 0; j < p.ni; ++j) d[p.s + i] += tin[(i / 4) * kLaneInF + 32 + 4 * j + i % 4] * pj[j];
                    }
                    if (last)
                        d[N] = s3 * (w[p.m - 1] + end.sE * we) + end.cs * ps + end.ce * pe +
                               (p.ni > 0 ? end.cj * pj[p.ni - 1] : 0.f);
                }
            }
        }
        double a = 0, b = 0;
        for (int i = 0; i <= N; ++i) { a += (d[i] - ref[i]) * (d[i] - ref[i]); b += ref[i] * ref[i]; }
        errs[along_x] = std::sqrt(a / b);
    }
    if (fails) return 1;
    std::printf("ok %.2e %.2e\n", errs[0], errs[1]);
    return 0;
}
