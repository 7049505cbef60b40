// Host FP64 tables of one axis: PMBC rows (paper Sec. 3.2, eq. PMBC and
// PMBC_coeffcients), row kinds, and the LU factors of the derivative systems.
//
// Rows of b = A^{-1} of the global natural-end collocation system (Sec. 3.1,
// eq. spline_cofficient_eq) are obtained from its reduction: the natural rows give
// v~_0 = v_0 and v~_N = v_N, the ghosts are v~_{-1} = 2 v~_0 - v~_1 and
// v~_{N+1} = 2 v~_N - v~_{N-1}, and the interior coefficients solve the symmetric
// Toeplitz system tridiag(1,4,1) v~ = 6 v - (boundary terms).  Row i of its inverse
// is one Thomas solve with the unit vector e_i.  The periodic line uses the
// circulant collocation system, whose inverse column has the closed form
// g_k = alpha (r^k + r^{N-k}), r = sqrt(3) - 2, from the two decaying homogeneous
// solutions of the three-term recurrence.
#include <algorithm>
#include <array>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <functional>
#include <map>

#include "loss_internal.h"
#include "tile_index.h"

namespace loss {
namespace {

// Solve tridiag(1,4,1) x = e_i of size n (unknowns 0..n-1), Thomas in FP64.
void toeplitz_unit_solve(int n, int i, std::vector<double> &x)
{
    std::vector<double> cpr(n), d(n, 0.0);
    x.assign(n, 0.0);
    d[i] = 1.0;
    double den = 4.0;
    cpr[0] = 1.0 / den;
    d[0] = d[0] / den;
    for (int k = 1; k < n; ++k) {
        den = 4.0 - cpr[k - 1];
        cpr[k] = 1.0 / den;
        d[k] = (d[k] - d[k - 1]) / den;
    }
    x[n - 1] = d[n - 1];
    for (int k = n - 2; k >= 0; --k) x[k] = d[k] - cpr[k] * x[k + 1];
}

// Row i (-1 <= i <= N+1) of b = A^{-1}, natural ends: out[k] = b_{i,k}, k = 0..N.
void natural_inverse_row(int N, int i, std::vector<double> &out)
{
    out.assign(N + 1, 0.0);
    if (i == 0) { out[0] = 1.0; return; }
    if (i == N) { out[N] = 1.0; return; }
    if (i == -1 || i == N + 1) {
        // ghost rows from the natural end rows
        int inner = (i == -1) ? 1 : N - 1, end = (i == -1) ? 0 : N;
        natural_inverse_row(N, inner, out);
        for (double &v : out) v = -v;
        out[end] += 2.0;
        return;
    }
    // interior: v~_i = sum_m G_{i,m} (6 v_m - [m=1] v_0 - [m=N-1] v_N), G = T^{-1},
    // T = tridiag(1,4,1) on nodes 1..N-1 (index m-1)
    std::vector<double> g;
    toeplitz_unit_solve(N - 1, i - 1, g);   // row i of G (G is symmetric)
    for (int m = 1; m <= N - 1; ++m) out[m] = 6.0 * g[m - 1];
    out[0] = -g[0];
    out[N] -= g[N - 2];
}

// First column of the circulant inverse (N distinct nodes).
void periodic_inverse_col(int N, std::vector<double> &g)
{
    const double r = std::sqrt(3.0) - 2.0;
    g.assign(N, 0.0);
    const double rN = std::pow(r, N), rN1 = std::pow(r, N - 1);
    const double alpha = 6.0 / (4.0 + 2.0 * r + 2.0 * rN1 + 4.0 * rN);
    for (int k = 0; k < N; ++k) g[k] = alpha * (std::pow(r, k) + std::pow(r, N - k));
}

// Rows of composition a chunk boundary needs in one sweep direction.  Forward
// elimination: y_r = rhs_r - f_r y_{r-1} on rows lo..hi-1 (the carry into row lo
// is exact).  The carry into row q depends on the one W rows earlier through the
// product f_{q-W} ... f_{q-1}; the window stops growing once it reaches row lo or
// that product is below tol.
int forward_reach(const std::vector<double> &f, int lo, int hi, double tol)
{
    int R = 0;
    for (int q = lo + 1; q < hi; ++q) {
        double prod = 1.0;
        int W = 0;
        while (q - W > lo && std::fabs(prod) > tol) { prod *= f[q - 1 - W]; ++W; }
        R = std::max(R, W);
    }
    return R;
}

// Back substitution: w_r = (y_r - g_r w_{r+1}) / d_r on rows lo..hi-1 (the carry
// into row hi-1 is the exact closing-row value).
int backward_reach(const std::vector<double> &g, int lo, int hi, double tol)
{
    int R = 0;
    for (int r = lo; r + 1 < hi; ++r) {
        double prod = 1.0;
        int W = 0;
        while (r + W + 1 < hi && std::fabs(prod) > tol) { prod *= g[r + 1 + W]; ++W; }
        R = std::max(R, W);
    }
    return R;
}

}  // namespace

std::string build_axis(AxisHost &ax, int N, double h, int M, int halo, int end_mode)
{
    if (N < 2) return "an axis needs at least 2 intervals";
    if (M < 1) return "patch length must be >= 1";
    if (halo < 1 || halo > kMaxHalo) return "halo must be in 1..64";
    if (!(h > 0.0)) return "spacing must be positive";
    if (end_mode == 2 && 2 * halo + 1 > N) return "periodic axis needs 2*halo+1 <= n";
    if (end_mode < 0 || end_mode > 2) return "unknown end mode";
    ax = AxisHost();
    ax.N = N; ax.M = M; ax.halo = halo; ax.end_mode = end_mode; ax.h = h;
    ax.p = (N + M - 1) / M;
    const int n = N + 1, ntap = 2 * halo + 1;
    ax.kind.assign(n, ROW_INTERIOR);
    for (int J = M; J < N; J += M) ax.kind[J] = ROW_JUNCTION;
    if (end_mode == 0) {
        ax.kind[0] = ROW_NATURAL_L;
        ax.kind[N] = ROW_NATURAL_R;
    } else {
        ax.kind[0] = ax.kind[N] = ROW_JUNCTION;
    }
    // ---- PMBC rows ------------------------------------------------------
    ax.slot.assign(n, -1);
    std::vector<double> rp, rm, g;
    if (end_mode == 2) periodic_inverse_col(N, g);
    for (int J = 0; J <= N; ++J) {
        if (ax.kind[J] != ROW_JUNCTION) continue;
        int s = (int)ax.junction_node.size();
        ax.slot[J] = s;
        ax.junction_node.push_back(J);
        ax.tap_idx.resize((size_t)(s + 1) * ntap, -1);
        ax.tap_c.resize((size_t)(s + 1) * ntap, 0.0);
        if (end_mode == 2) {
            for (int t = 0; t < ntap; ++t) {
                int k = ((J - halo + t) % N + N) % N;
                int ip = ((J + 1 - k) % N + N) % N, im = ((J - 1 - k) % N + N) % N;
                ax.tap_idx[(size_t)s * ntap + t] = k;
                ax.tap_c[(size_t)s * ntap + t] = (g[ip] - g[im]) / (2.0 * h);
            }
        } else {
            natural_inverse_row(N, J + 1, rp);
            natural_inverse_row(N, J - 1, rm);
            for (int t = 0; t < ntap; ++t) {
                int k = J - halo + t;
                if (k < 0 || k > N) continue;
                ax.tap_idx[(size_t)s * ntap + t] = k;
                ax.tap_c[(size_t)s * ntap + t] = (rp[k] - rm[k]) / (2.0 * h);
            }
        }
    }
    // ---- rows of T and G ---------------------------------------------------
    ax.sub.assign(n, 0.0); ax.diag.assign(n, 0.0); ax.sup.assign(n, 0.0);
    ax.cm.assign(n, 0.0); ax.c0.assign(n, 0.0); ax.cp.assign(n, 0.0);
    const double s3 = 3.0 / h;
    for (int i = 0; i <= N; ++i) {
        switch (ax.kind[i]) {
        case ROW_INTERIOR:
            ax.sub[i] = 1.0; ax.diag[i] = 4.0; ax.sup[i] = 1.0;
            ax.cm[i] = -s3; ax.cp[i] = s3;
            break;
        case ROW_JUNCTION:
            ax.diag[i] = 1.0;
            break;
        case ROW_NATURAL_L:
            ax.diag[i] = 2.0; ax.sup[i] = 1.0;
            ax.c0[i] = -s3; ax.cp[i] = s3;
            break;
        case ROW_NATURAL_R:
            ax.sub[i] = 1.0; ax.diag[i] = 2.0;
            ax.cm[i] = -s3; ax.c0[i] = s3;
            break;
        }
    }
    // ---- LU of T, no pivoting ---------------------------------------------
    ax.m.assign(n, 0.0); ax.invd.assign(n, 0.0);
    double dprev = 0.0;
    for (int i = 0; i <= N; ++i) {
        double mi = (i == 0) ? 0.0 : ax.sub[i] / dprev;
        double di = ax.diag[i] - (i == 0 ? 0.0 : mi * ax.sup[i - 1]);
        ax.m[i] = mi;
        ax.invd[i] = 1.0 / di;
        dprev = di;
    }
    // ---- LU of T^T ---------------------------------------------------------
    ax.mT.assign(n, 0.0); ax.invdT.assign(n, 0.0); ax.supT.assign(n, 0.0); ax.subT.assign(n, 0.0);
    dprev = 0.0;
    for (int i = 0; i <= N; ++i) {
        double subT = (i == 0) ? 0.0 : ax.sup[i - 1];
        double supT = (i == N) ? 0.0 : ax.sub[i + 1];
        double mi = (i == 0) ? 0.0 : subT / dprev;
        double di = ax.diag[i] - (i == 0 ? 0.0 : mi * ax.supT[i - 1]);
        ax.subT[i] = subT;
        ax.supT[i] = supT;
        ax.mT[i] = mi;
        ax.invdT[i] = 1.0 / di;
        dprev = di;
    }
    // ---- transposed PMBC gather ---------------------------------------------
    // (a halo wider than the patches reaches a node from several junction rows: the
    // table is as wide as the most rows reaching one node)
    std::vector<int> cnt(n, 0);
    for (size_t s = 0; s < ax.junction_node.size(); ++s)
        for (int t = 0; t < ntap; ++t) {
            const int k = ax.tap_idx[s * ntap + t];
            if (k >= 0 && ax.tap_c[s * ntap + t] != 0.0) ++cnt[k];
        }
    ax.gmax = std::max(1, *std::max_element(cnt.begin(), cnt.end()));
    ax.g_node.assign((size_t)n * ax.gmax, -1);
    ax.g_c.assign((size_t)n * ax.gmax, 0.0);
    std::fill(cnt.begin(), cnt.end(), 0);
    for (size_t s = 0; s < ax.junction_node.size(); ++s) {
        for (int t = 0; t < ntap; ++t) {
            int k = ax.tap_idx[s * ntap + t];
            if (k < 0) continue;
            double c = ax.tap_c[s * ntap + t];
            if (c == 0.0) continue;
            ax.g_node[(size_t)k * ax.gmax + cnt[k]] = ax.junction_node[s];
            ax.g_c[(size_t)k * ax.gmax + cnt[k]] = c;
            ++cnt[k];
        }
    }
    // ---- second-derivative system, patch by patch ---------------------------
    // first row: Hermite [2,1] at a junction, identity (s'' = 0) at a natural end;
    // interior rows [1,4,1]; closing row: Hermite [1,2] or identity.
    ax.m2.assign(n, 0.0); ax.invd2.assign(n, 0.0); ax.sup2.assign(n, 0.0);
    ax.m2c.assign(n, 0.0); ax.invd2c.assign(n, 0.0);
    for (int l = 0; l < ax.p; ++l) {
        int s = l * M, e = std::min(s + M, N);
        bool nat_l = ax.kind[s] == ROW_NATURAL_L, nat_r = ax.kind[e] == ROW_NATURAL_R;
        double d = nat_l ? 1.0 : 2.0;
        double supprev = nat_l ? 0.0 : 1.0;
        ax.m2[s] = 0.0; ax.invd2[s] = 1.0 / d; ax.sup2[s] = supprev;
        for (int i = s + 1; i < e; ++i) {
            double mi = 1.0 / d;
            d = 4.0 - mi * supprev;
            ax.m2[i] = mi; ax.invd2[i] = 1.0 / d; ax.sup2[i] = 1.0;
            supprev = 1.0;
        }
        if (nat_r) {
            ax.m2c[e] = 0.0; ax.invd2c[e] = 1.0;
        } else {
            double mi = 1.0 / d;
            ax.m2c[e] = mi;
            ax.invd2c[e] = 1.0 / (2.0 - mi * supprev);
        }
    }
    // ---- carry reach over the three systems, both sweeps ---------------------
    std::vector<double> g1(n), gT(n), g2(n);
    for (int i = 0; i < n; ++i) {
        g1[i] = ax.sup[i] * ax.invd[i];
        gT[i] = ax.supT[i] * ax.invdT[i];
        g2[i] = ax.sup2[i] * ax.invd2[i];
    }
    ax.reach = 1;
    for (int l = 0; l < ax.p; ++l) {
        int s = l * M, e = std::min(s + M, N);
        for (const std::vector<double> *f : {&ax.m, &ax.mT, &ax.m2})
            ax.reach = std::max(ax.reach, forward_reach(*f, s, e, kReachTol));
        for (const std::vector<double> *g : {&g1, &gT, &g2})
            ax.reach = std::max(ax.reach, backward_reach(*g, s, e, kReachTol));
    }
    return std::string();
}

namespace {

// Row J of the order-1 or order-2 derivative operator of the patch [s, e] of an axis as a
// tap row: z with T^T z = e_J on the patch (T the slope or the moment system), then z^T G.
// J is far enough inside the patch for the end rows' own right-hand sides to enter below
// the tolerance.
void interior_row(const AxisHost &ax, int order, int s, int e, int J, std::vector<double> &row)
{
    const int n = e - s + 1;
    std::vector<double> diag(n, 4.0), sub(n, 1.0), sup(n, 1.0);
    for (int i : {0, n - 1}) {
        const int k = i ? e : s;
        const bool nat = ax.kind[k] == ROW_NATURAL_L || ax.kind[k] == ROW_NATURAL_R;
        diag[i] = order == 1 ? (nat ? 2.0 : 1.0) : (nat ? 1.0 : 2.0);
        if (order == 1 ? !nat : nat) sub[i] = sup[i] = 0.0;   // identity row
    }
    std::vector<double> cp(n), z(n, 0.0);
    z[J - s] = 1.0;
    // Thomas on T^T: sub-diagonal sup[i-1], super-diagonal sub[i+1]
    double den = diag[0];
    cp[0] = (n > 1 ? sub[1] : 0.0) / den;
    z[0] /= den;
    for (int i = 1; i < n; ++i) {
        const double lo = sup[i - 1];
        den = diag[i] - lo * cp[i - 1];
        cp[i] = (i + 1 < n ? sub[i + 1] : 0.0) / den;
        z[i] = (z[i] - lo * z[i - 1]) / den;
    }
    for (int i = n - 2; i >= 0; --i) z[i] -= cp[i] * z[i + 1];
    row.assign(n, 0.0);
    const double w1 = 3.0 / ax.h, w2 = 6.0 / (ax.h * ax.h);
    for (int i = 1; i + 1 < n; ++i) {
        row[i - 1] += z[i] * (order == 1 ? -w1 : w2);
        row[i] += z[i] * (order == 1 ? 0.0 : -2.0 * w2);
        row[i + 1] += z[i] * (order == 1 ? w1 : w2);
    }
}

// Elimination rows of a piece: y_i = nf y_{i-1} + sc (right-hand side), w_i = fi y_i + g
// w_{i+1}; rows past the piece pass the carries on.
struct Row {
    double nf = 1.0, sc = 0.0, fi = 0.0, g = 1.0;
};

typedef std::vector<double> V;

// First (at_end false) or last (true) row of the inverse of a piece's interior system of
// T^T: [1 4 1] rows s+1 .. e-1, and the rows of a natural end.  row[k] belongs to node lo + k.
void interior_inverse_end(const AxisHost &ax, int s, int e, bool at_end, int &lo, std::vector<double> &row)
{
    lo = ax.kind[s] == ROW_NATURAL_L ? s : s + 1;
    const int hi = ax.kind[e] == ROW_NATURAL_R ? e : e - 1;
    const int n = hi - lo + 1;
    row.assign(std::max(n, 0), 0.0);
    if (n < 1) return;
    auto diag = [&](int i) { return lo + i == s || lo + i == e ? 2.0 : 4.0; };
    std::vector<double> cp(n);
    row[at_end ? n - 1 : 0] = 1.0;
    double den = diag(0);
    cp[0] = 1.0 / den;
    row[0] /= den;
    for (int i = 1; i < n; ++i) {
        den = diag(i) - cp[i - 1];
        cp[i] = 1.0 / den;
        row[i] = (row[i] - row[i - 1]) / den;
    }
    for (int i = n - 2; i >= 0; --i) row[i] -= cp[i] * row[i + 1];
}

}  // namespace

std::string build_tile(const AxisHost &ax, bool along_x, int op, bool across, TileHost &t)
{
    t = TileHost();
    const int N = ax.N;
    if (ax.halo > kTileHalo) return "halo wider than the tile window";
    const double s3 = 3.0 / ax.h, w2 = 6.0 / (ax.h * ax.h);
    const int nt = 2 * ax.halo + 1;
    // ---- pieces: at most kTileM intervals; along x the closing node of the line takes a lane
    // of the last one -------------------------------------------------------------------------
    std::vector<int> jn;                // junctions and ends
    for (int l = 0; l <= ax.p; ++l) jn.push_back(std::min(l * ax.M, N));
    const int end_cap = along_x ? kTileM - 1 : kTileM;
    if (!across) {
        // Between junctions: patches longer than a piece are cut evenly; along x the cuts fall
        // on multiples of 16 nodes, so that a tile's rows start on 64-byte boundaries where the
        // patches do (a row start inside a 64-byte sector costs a partial write).
        for (int l = 0; l < ax.p; ++l) {
            const int s = jn[l], e = jn[l + 1], m = e - s;
            const int cap = e == N ? end_cap : kTileM;
            const int n = (m + cap - 1) / cap;
            std::vector<int> cut(n + 1);
            for (int i = 0; i <= n; ++i) cut[i] = (int)((int64_t)i * m / n);
            if (along_x) {
                std::vector<int> al = cut;
                bool ok = true;
                for (int i = 1; i < n; ++i) al[i] = (cut[i] + 8) / 16 * 16;
                for (int i = 0; i < n; ++i) ok = ok && al[i + 1] > al[i] && al[i + 1] - al[i] <= (i == n - 1 ? cap : kTileM);
                // taps at a cut need its distance to the patch ends (kTileHalo) as an equal cut has it
                if (ok && (n == 1 || (al[1] > kTileHalo && m - al[n - 1] > kTileHalo))) cut = al;
            }
            for (int i = 0; i < n; ++i) t.sb.push_back(s + cut[i]);
        }
        t.sb.push_back(N);
    } else {
        // Across junctions (slopes of patches shorter than a piece; moments are two-valued at a
        // junction): the fewest pieces that end on junctions or on cuts at least kCutGap inside a
        // patch and hold at most kTileIn junctions, of which the middle ones' taps stay inside;
        // then few junctions inside, starts on multiples of 16 along x, even lengths.  Along the
        // rows the longest piece is as short as their number allows (waves per workgroup).
        if (op == TILE_D2 || ax.M < kTileInGap || ax.M >= kTileM || ax.p < 2) return "no pieces across junctions";
        auto split = [&](int cap, std::vector<int> &out) {
            const int64_t inf = int64_t(1) << 60;
            std::vector<int64_t> f(N + 1, inf);
            std::vector<int> from(N + 1, -1);
            f[0] = 0;
            for (int e = 1; e <= N; ++e) {
                const int l = (e - 1) / ax.M, ps = jn[l], pe = jn[l + 1];
                if (e != pe && (e - ps < kCutGap || pe - e < kCutGap)) continue;
                for (int s = std::max(0, e - std::min(cap, e == N ? end_cap : kTileM)); s < e; ++s) {
                    if (f[s] >= inf) continue;
                    const int j0 = s / ax.M + 1, j1 = l;         // junctions inside: j0 .. j1 times M
                    const int ni = std::max(0, j1 - j0 + 1);
                    if (ni > kTileIn) continue;
                    bool ok = true;
                    for (int j = j0 + 1; j < j1; ++j) ok = ok && j * ax.M - ax.halo >= s && j * ax.M + ax.halo <= e;
                    if (!ok) continue;
                    const int64_t c = f[s] + 100000000 + 100000 * ni + (along_x && s % 16 ? 3000 : 0) + (e - s) * (e - s) / 64;
                    if (c < f[e]) {
                        f[e] = c;
                        from[e] = s;
                    }
                }
            }
            out.clear();
            if (f[N] >= inf) return;
            for (int e = N; e > 0; e = from[e]) out.push_back(e);
            out.push_back(0);
            std::reverse(out.begin(), out.end());
        };
        auto inside_count = [&](const std::vector<int> &v) {
            return std::count_if(jn.begin(), jn.end(), [&](int J) { return !std::binary_search(v.begin(), v.end(), J); });
        };
        split(kTileM, t.sb);
        if (t.sb.empty()) return "no split into tile pieces";
        for (int cap = kTileM - kTileC; !along_x && cap >= kTileC; cap -= kTileC) {
            std::vector<int> even;
            split(cap, even);
            if (even.size() != t.sb.size() || inside_count(even) > inside_count(t.sb)) break;
            t.sb = even;
        }
    }
    t.nsub = (int)t.sb.size() - 1;
    if (along_x) {
        t.lanes.reserve((size_t)t.nsub * 16 * kLaneF);
        t.lanes_in.reserve((size_t)t.nsub * 16 * kLaneInF);
    } else {
        t.chunk.reserve((size_t)t.nsub * kTileWaves * kChunkF);
    }
    t.halo_c.reserve((size_t)t.nsub * kTapW * 4);
    // ---- their ends and the junctions inside, with their tap rows (order-1 slopes; order 2 of
    // a cut), in the order of the line ---------------------------------------------------------
    std::vector<int> sb, bh;
    std::vector<double> taps;
    std::vector<char> real;             // a junction or an end of the method's patches
    std::map<std::array<int, 4>, std::vector<double>> rows;
    std::set_union(jn.begin(), jn.end(), t.sb.begin(), t.sb.end(), std::back_inserter(sb));
    for (int J : sb) {
        const size_t o = taps.size();
        taps.resize(o + kTapW, 0.0);
        real.push_back(J % ax.M == 0 || J == N);
        if (ax.slot[J] >= 0) {
            bh.push_back(ax.halo);
            for (int k = 0; k < nt; ++k) taps[o + k] = ax.tap_c[(size_t)ax.slot[J] * nt + k];
        } else if (real.back()) {
            bh.push_back(0);
        } else {
            const int s = J / ax.M * ax.M, e = std::min(s + ax.M, N);
            // equal for equal patches
            const std::array<int, 4> key = {J - s, e - s, ax.kind[s], ax.kind[e]};
            auto known = rows.find(key);
            if (known == rows.end()) {
                known = rows.emplace(key, std::vector<double>()).first;
                interior_row(ax, op == TILE_D2 ? 2 : 1, s, e, J, known->second);
            }
            const std::vector<double> &row = known->second;
            int H = kTileHalo;
            auto mag = [&](int d) {
                const int a = J - d - s, b = J + d - s;
                return std::max(a >= 0 ? std::fabs(row[a]) : 0.0, b <= e - s ? std::fabs(row[b]) : 0.0);
            };
            while (H > 1 && mag(H) <= kTapTol * (op == TILE_D2 ? w2 : s3)) --H;
            bh.push_back(H);
            for (int d = -H; d <= H; ++d)
                if (J + d >= s && J + d <= e) taps[o + H + d] = row[J + d - s];
        }
    }
    auto index_of = [&](int J) { return (int)(std::lower_bound(sb.begin(), sb.end(), J) - sb.begin()); };
    if (op == TILE_DT) {
        if (ax.end_mode == 2) return "transposed taps wrap around a periodic line";
        // a node takes the transposed taps of its own piece's junctions only
        for (size_t b = 0; b < sb.size(); ++b)
            for (int w = 0; w < t.nsub; ++w) {
                if (sb[b] >= t.sb[w] && sb[b] <= t.sb[w + 1]) continue;
                const int last = w == t.nsub - 1 ? N : t.sb[w + 1] - 1;
                for (int d = -bh[b]; d <= bh[b] && bh[b] > 0; ++d)
                    if (taps[b * kTapW + bh[b] + d] != 0.0 && sb[b] + d >= t.sb[w] && sb[b] + d <= last)
                        return "transposed taps reach past the neighbouring piece";
            }
    }
    for (int w0 = 0; w0 < t.nsub; ++w0) {
        const int s = t.sb[w0], e = t.sb[w0 + 1], m = e - s;
        const int b = index_of(s), be = index_of(e), ni = be - b - 1;   // b + 1 .. be - 1: inside
        t.max_m = std::max(t.max_m, m);
        const bool nat_s = ax.kind[s] == ROW_NATURAL_L, nat_e = ax.kind[e] == ROW_NATURAL_R;
        const double *cs = &taps[(size_t)b * kTapW], *ce = &taps[(size_t)be * kTapW];
        auto tap = [](const double *c, int H, int J, int k) {
            const int d = k - (J - H);
            return d >= 0 && d <= 2 * H ? c[d] : 0.0;
        };
        // taps of the start and the closing right-hand side at node k, and how far they reach
        // outside the piece
        int hs = bh[b], he = bh[be], hi[kTileIn] = {};
        std::function<double(int)> tap_s = [&](int k) { return tap(cs, hs, s, k); };
        std::function<double(int)> tap_e = [&](int k) { return tap(ce, he, e, k); };
        std::function<double(int)> tap_j[kTileIn];
        for (int j = 0; j < ni; ++j) {
            const int J = sb[b + 1 + j];
            const double *cj = &taps[(size_t)(b + 1 + j) * kTapW];
            hi[j] = bh[b + 1 + j];
            tap_j[j] = [=](int k) { return tap(cj, hi[j], J, k); };
        }
        auto inside = [&](int i) {      // the junction inside at node s + i, or -1
            for (int j = 0; j < ni; ++j)
                if (sb[b + 1 + j] == s + i) return j;
            return -1;
        };
        std::vector<Row> r(kTileM);
        double iE = 1.0, imE = 0.0, sE = 0.0, endc = 0.0, endd = 0.0;
        double d = 0.0, sup = 0.0;
        V as, ae;                       // TILE_DT: transposed-system taps of y_s, y_e by node offset
        if (op == TILE_D1) {
            for (int i = 0; i < m; ++i) {
                if (i == 0) {           // junction: the slope is the carry; natural end row
                    d = nat_s ? 2.0 : 1.0;
                    sup = nat_s ? 1.0 : 0.0;
                    r[0] = nat_s ? Row{0.0, s3, 0.5, -0.5} : Row{1.0, 0.0, 1.0, 0.0};
                } else if (inside(i) >= 0) {   // the slope enters as p_m
                    d = 1.0;
                    sup = 0.0;
                    r[i] = Row{0.0, 0.0, 1.0, 0.0};
                } else {
                    const double mi = 1.0 / d;
                    d = 4.0 - mi * sup;
                    sup = 1.0;
                    r[i] = Row{-mi, s3, 1.0 / d, -1.0 / d};
                }
            }
            if (nat_e) {
                const double mi = 1.0 / d, de = 2.0 - mi * sup;
                iE = 1.0 / de;
                imE = mi / de;
                sE = s3;
            }
        } else if (op == TILE_D2) {
            // moments: Hermite rows at a junction (the slope enters the first row with -6/h,
            // the closing one with 6/h), zero at a natural end, the tapped moment at a cut
            for (int i = 0; i < m; ++i) {
                if (i == 0) {
                    const bool herm = real[b] && !nat_s;
                    d = herm ? 2.0 : 1.0;
                    sup = herm ? 1.0 : 0.0;
                    r[0] = herm ? Row{-6.0 / ax.h, w2, 0.5, -0.5} : Row{nat_s ? 0.0 : 1.0, 0.0, 1.0, 0.0};
                } else {
                    const double mi = 1.0 / d;
                    d = 4.0 - mi * sup;
                    sup = 1.0;
                    r[i] = Row{-mi, w2, 1.0 / d, -1.0 / d};
                }
            }
            if (nat_e) {
                iE = 0.0;
            } else if (real[be]) {
                const double mi = 1.0 / d, de = 2.0 - mi * sup;
                iE = 1.0 / de;
                imE = mi / de;
                sE = -w2;
                tap_e = [&](int k) { return 6.0 / ax.h * tap(ce, he, e, k); };
            }
        } else {
            // T^T on the piece's interior rows; the junction rows follow from the neighbouring
            // interior values: y_J = z_J - y_{J-1} - y_{J+1}, here as taps
            for (int i = nat_s ? 0 : 1; i < m; ++i) {
                if (inside(i) >= 0) {
                    r[i] = Row{0.0, 0.0, 0.0, 0.0};
                    continue;
                }
                const bool first = i == (nat_s ? 0 : 1) || inside(i - 1) >= 0;
                const double mi = first ? 0.0 : 1.0 / d;
                d = first ? (nat_s && i == 0 ? 2.0 : 4.0) : 4.0 - mi;
                r[i] = Row{-mi, 1.0, 1.0 / d, -1.0 / d};
            }
            if (!nat_s) r[0] = Row{0.0, 0.0, 0.0, 0.0};
            iE = 0.0;
            if (nat_e) {
                const bool any = m > (nat_s ? 0 : 1) && inside(m - 1) < 0;
                const double mi = any ? 1.0 / d : 0.0, de = 2.0 - mi;
                iE = 1.0 / de;
                imE = mi / de;
            }
            auto end_taps = [&](int J, V &a) {      // a[kTileHalo + offset]
                a.assign(2 * kTileHalo + 1, 0.0);
                a[kTileHalo] = 1.0;
                const int j = index_of(J);
                int reach = 0;
                for (int side = 0; side < 2; ++side) {
                    const int p = side ? j : j - 1; // the piece right or left of J
                    if (p < 0 || p + 1 >= (int)sb.size()) continue;
                    int lo;
                    std::vector<double> row;
                    interior_inverse_end(ax, sb[p], sb[p + 1], side == 0, lo, row);
                    for (int k = 0; k < (int)row.size(); ++k) {
                        const int off = lo + k - J;
                        if (std::abs(off) <= kTileHalo && std::fabs(row[k]) > kTapTol) {
                            a[kTileHalo + off] -= row[k];
                            reach = std::max(reach, std::abs(off));
                        }
                    }
                }
                return reach;
            };
            hs = he = 0;
            if (!nat_s) hs = end_taps(s, as);
            if (!nat_e) he = end_taps(e, ae);
            tap_s = [&](int k) { return !nat_s && std::abs(k - s) <= kTileHalo ? as[kTileHalo + k - s] : 0.0; };
            tap_e = [&](int k) { return nat_e ? (k == e ? 1.0 : 0.0)
                                              : (std::abs(k - e) <= kTileHalo ? ae[kTileHalo + k - e] : 0.0); };
            for (int j = 0; j < ni; ++j) {
                const int J = sb[b + 1 + j];
                V aj;
                hi[j] = end_taps(J, aj);
                tap_j[j] = [=](int k) { return std::abs(k - J) <= kTileHalo ? aj[kTileHalo + k - J] : 0.0; };
            }
            sE = nat_e ? 1.0 : 0.0;
            endc = tap(cs, bh[b], s, e);            // transposed PMBC taps at the closing node
            endd = nat_e ? 0.0 : tap(ce, bh[be], e, e);
        }
        if (op != TILE_DT) {            // sums of the tap rows
            for (int k = s - kTileHalo; k <= s + kTileHalo; ++k) endc += tap_s(k);
            for (int k = e - kTileHalo; k <= e + kTileHalo; ++k) endd += tap_e(k);
        }
        int hl = std::max(hs, he - m), hr = std::max(he, hs - m), hin = 0;
        for (int j = 0; j < ni; ++j) {
            const int J = sb[b + 1 + j];
            if ((j == 0 || j == ni - 1)) {
                hl = std::max(hl, hi[j] - (J - s));
                hr = std::max(hr, hi[j] - (e - J));
            } else if (hi[j] > J - s || hi[j] > e - J) {
                return "taps of a middle junction leave the piece";
            }
            hin = std::max(hin, hi[j]);
        }
        const int pz = hs | he << 8 | hl << 16 | hr << 24, pw = ni | hin << 8;
        const Piece p = make_piece(s, e, pz, pw);
        for (int v : {s, e, pz, pw}) t.piece.push_back(v);
        double endj = 0.0;              // transposed: what node N takes from the last junction inside
        for (int j = 0; j < ni && op == TILE_DT && e == N; ++j) {
            endj = tap(&taps[(size_t)(b + 1 + j) * kTapW], bh[b + 1 + j], sb[b + 1 + j], e);
            if (j < ni - 1 && endj != 0.0) return "transposed taps of several junctions reach the last node";
        }
        for (double v : {iE, imE, sE, endj, endc, endd, nat_s ? -1.0 : 0.0, 0.0}) t.ends.push_back((float)v);
        for (int i = 0; i < kTapW; ++i) {
            const bool in = i < halo_count(p);
            const int k = in ? halo_pos(p, i) : e;
            t.halo_node.push_back(line_node(k, N, ax.end_mode == 2));
            const bool real_node = ax.end_mode == 2 || (k >= 0 && k <= N);
            t.halo_c.push_back(in && real_node ? (float)tap_s(k) : 0.f);
            t.halo_c.push_back(in && real_node ? (float)tap_e(k) : 0.f);
            t.halo_c.push_back(in && real_node && ni > 0 ? (float)tap_j[0](k) : 0.f);
            t.halo_c.push_back(in && real_node && ni > 1 ? (float)tap_j[ni - 1](k) : 0.f);
        }
        auto push = [&](std::vector<float> &v, double x) { v.push_back((float)x); };
        auto push_bits = [&](std::vector<float> &v, int x) {
            float f;
            std::memcpy(&f, &x, 4);
            v.push_back(f);
        };
        if (!along_x) {
            // strided passes: the carries of the chunks of kTileC rows as sums over the chunks'
            // own results.  B_j: chunk j eliminated from a zero carry; W_j: its back
            // substitution from zero carries; p_0: the start junction's value; p_1: the closing
            // row's right-hand side; p_2 ..: the junctions inside.  Vectors over (B_0.., W_0.., p_0..).
            constexpr int nw = kTileWaves, np = 2 * nw, nv = np + 2 + kTileIn;
            const int nch = (m + kTileC - 1) / kTileC;
            std::vector<V> yin(nw + 1, V(nv, 0.0)), win(nw, V(nv, 0.0)), prev(nw, V(nv, 0.0));
            std::vector<double> A(nw, 1.0), Q(nw, 1.0), R(nw, 0.0), Rm(nw, 0.0);
            std::vector<int> cm(nw, -1);                 // the chunk's junction inside
            std::vector<V> qm(nw, V(kTileC, 0.0));       // its rows' response to it
            if (op != TILE_DT) yin[0][np] = 1.0;
            for (int w = 0; w < nch; ++w) {
                double back[kTileC];
                for (int c = 0; c < kTileC; ++c) {
                    const Row &q = r[w * kTileC + c];
                    A[w] *= q.nf;
                    back[c] = A[w];
                    Q[w] *= q.g;
                    const int j = op == TILE_DT ? -1 : inside(w * kTileC + c);
                    if (j >= 0) cm[w] = j;
                    qm[w][c] = j >= 0 ? 1.0 : (c > 0 ? q.nf * qm[w][c - 1] : 0.0);
                }
                for (int c = kTileC - 1; c >= 0; --c) {
                    const Row &q = r[w * kTileC + c];
                    R[w] = q.fi * back[c] + q.g * R[w];
                    Rm[w] = q.fi * qm[w][c] + q.g * Rm[w];
                }
                for (int k = 0; k < nv; ++k) yin[w + 1][k] = A[w] * yin[w][k];
                yin[w + 1][w] += 1.0;
                if (cm[w] >= 0) yin[w + 1][np + 2 + cm[w]] += qm[w][kTileC - 1];
            }
            for (int k = 0; k < nv; ++k) win[nch - 1][k] = -imE * yin[nch][k];
            win[nch - 1][np + 1] += iE;
            for (int w = nch - 2; w >= 0; --w) {
                for (int k = 0; k < nv; ++k) win[w][k] = R[w + 1] * yin[w + 1][k] + Q[w + 1] * win[w + 1][k];
                win[w][nw + w + 1] += 1.0;
                if (cm[w + 1] >= 0) win[w][np + 2 + cm[w + 1]] += Rm[w + 1];
            }
            for (int w = 1; w < nch; ++w) {             // the solution at the row before chunk w
                const Row &q = r[w * kTileC - 1];
                for (int k = 0; k < nv; ++k) prev[w][k] = q.fi * yin[w][k] + q.g * win[w - 1][k];
            }
            // the junctions around each chunk: the sums above involve no others
            std::vector<int> cl(nw, 0), cr(nw, 1);
            for (int j = 0; j < ni && op != TILE_DT; ++j)
                for (int w = 0; w < nch; ++w) {
                    const int i = sb[b + 1 + j] - s;
                    if (i < w * kTileC) cl[w] = 2 + j;
                    if (i >= (w + 1) * kTileC && cr[w] == 1) cr[w] = 2 + j;
                }
            for (int w = 0; w < nw; ++w) {
                const bool on = w < nch;
                const Row *q = &r[w * kTileC];
                double a = 1.0;
                for (int c = 0; c < kTileC; ++c) { a *= q[c].nf; push(t.chunk, on ? a : 0.0); }
                for (int j = 0; j < nw; ++j) push(t.chunk, on ? yin[w][j] : 0.0);
                for (int j = 0; j < nw; ++j) push(t.chunk, on ? win[w][j] : 0.0);
                for (int j = 0; j < nw; ++j) push(t.chunk, on ? win[w][nw + j] : 0.0);
                const int il = np + cl[w], im = cm[w] >= 0 ? np + 2 + cm[w] : il, ir = np + cr[w];
                for (double v : {yin[w][il], win[w][im], win[w][ir], prev[w][np + 1]}) push(t.chunk, on ? v : 0.0);
                for (int k = np; k < nv && on; ++k)
                    if ((k != il && yin[w][k] != 0.0) || (k != im && k != ir && win[w][k] != 0.0)) return "carries of a chunk";
                for (int c = 0; c < kTileC; ++c) push(t.chunk, q[c].nf);
                for (int c = 0; c < kTileC; ++c) push(t.chunk, q[c].sc);
                for (int c = 0; c < kTileC; ++c) push(t.chunk, q[c].fi);
                for (int c = 0; c < kTileC; ++c) push(t.chunk, q[c].g);
                bool any[2] = {false, false};
                for (int k = 0; k < 2; ++k)
                    for (int c = 0; c < kTileC; ++c) {
                        const int i = s + w * kTileC + c;
                        const double v = i >= e ? 0.0 : (k ? tap_e(i) : tap_s(i));
                        any[k] = any[k] || v != 0.0;
                        push(t.chunk, v);
                    }
                for (int k = 0; k < 2; ++k) push(t.chunk, any[k] ? 1.0 : 0.0);
                // transposed: what the row takes from y_s and y_e
                bool anyc[2] = {false, false};
                float cc[2][kTileC];
                for (int k = 0; k < 2; ++k)
                    for (int c = 0; c < kTileC; ++c) {
                        const int i = s + w * kTileC + c;
                        const double v = op != TILE_DT || i >= e ? 0.0 : (k ? tap(ce, bh[be], e, i) : tap(cs, bh[b], s, i));
                        cc[k][c] = (float)v;
                        anyc[k] = anyc[k] || v != 0.0;
                    }
                for (int k = 0; k < 2; ++k) push(t.chunk, anyc[k] ? 1.0 : 0.0);
                for (int k = 0; k < 2; ++k)
                    for (int c = 0; c < kTileC; ++c) t.chunk.push_back(cc[k][c]);
                for (int j = 0; j < nw; ++j) push(t.chunk, prev[w][j]);
                for (int j = 0; j < nw; ++j) push(t.chunk, prev[w][nw + j]);
                float in[2][kTileIn][kTileC] = {};
                int any_in = 0;
                for (int j = 0; j < ni; ++j)
                    for (int c = 0; c < kTileC; ++c) {
                        const int i = s + w * kTileC + c;
                        if (i >= e) continue;
                        in[0][j][c] = (float)tap_j[j](i);
                        if (op == TILE_DT) in[1][j][c] = (float)tap(&taps[(size_t)(b + 1 + j) * kTapW], bh[b + 1 + j], sb[b + 1 + j], i);
                        any_in |= in[0][j][c] != 0.f || in[1][j][c] != 0.f;
                    }
                for (int v : {cl[w], cm[w] >= 0 ? 2 + cm[w] : -1, cr[w], any_in}) push_bits(t.chunk, v);
                for (int c = 0; c < kTileC; ++c) push(t.chunk, qm[w][c]);
                for (int k = 0; k < 2; ++k)
                    for (int j = 0; j < kTileIn; ++j)
                        for (int c = 0; c < kTileC; ++c) t.chunk.push_back(in[k][j][c]);
            }
        } else {
            // x pass: 16 lanes of four nodes.  The carries are composed in three doubling steps
            // whose multipliers do not depend on the data: lane 0 absorbs the slope, the
            // closing lane and those after it the closing value.
            constexpr int nl = kTileM / 4;
            const int kc = (m - 1) / 4;
            std::vector<double> a1(nl), b1(nl), qt(nl);
            double a0 = 0.0;
            for (int k = 0; k < nl; ++k) {
                double a = 1.0, q = 1.0;
                for (int c = 0; c < 4; ++c) { a *= r[4 * k + c].nf; q *= r[4 * k + c].g; }
                if (k == 0) a0 = a;
                a1[k] = k == 0 ? 0.0 : a;
                qt[k] = q;
                b1[k] = k >= kc ? 0.0 : q;
            }
            auto up = [&](const std::vector<double> &v, int k, int w) {   // product over lanes k, k-1, .. k-w+1
                double p = 1.0;
                for (int i = 0; i < w; ++i) p *= k - i >= 0 ? v[k - i] : 0.0;
                return p;
            };
            auto dn = [&](const std::vector<double> &v, int k, int w) {
                double p = 1.0;
                for (int i = 0; i < w; ++i) p *= k + i < nl ? v[k + i] : 0.0;
                return p;
            };
            for (int k = 0; k < nl; ++k) {
                for (int c = 0; c < 4; ++c) push(t.lanes, r[4 * k + c].nf);
                for (int c = 0; c < 4; ++c) push(t.lanes, r[4 * k + c].sc);
                for (int c = 0; c < 4; ++c) push(t.lanes, r[4 * k + c].fi);
                for (int c = 0; c < 4; ++c) push(t.lanes, r[4 * k + c].g);
                double a = 1.0;
                for (int c = 0; c < 4; ++c) { a *= r[4 * k + c].nf; push(t.lanes, a); }
                for (double v : {a1[k], up(a1, k, 2), up(a1, k, 4), k == 0 ? a0 : 0.0}) push(t.lanes, v);
                for (double v : {b1[k], dn(b1, k, 2), dn(b1, k, 4), k == kc ? qt[k] : (k > kc ? 1.0 : 0.0)}) push(t.lanes, v);
                // taps k, k + 16, k + 32 of a junction and their places in the LDS row, byte offsets
                auto put_taps = [&](std::vector<float> &v, const std::function<double(int)> &f, int H, int d0) {
                    float cf[3];
                    int pos[3];
                    for (int h = 0; h < 3; ++h) {
                        const int i = k + 16 * h;
                        const bool in = i <= 2 * H;
                        const int node = s + d0 + i;
                        const bool real_node = ax.end_mode == 2 || (node >= 0 && node <= N);
                        cf[h] = in && real_node ? (float)f(node) : 0.f;
                        pos[h] = 4 * tap_slot(p, d0 + (in ? i : 0));
                    }
                    for (float x : {cf[0], cf[1], cf[2], 0.f}) v.push_back(x);
                    for (int x : {pos[0], pos[1], pos[2], 0}) push_bits(v, x);
                };
                put_taps(t.lanes, tap_s, p.hs, -p.hs);
                put_taps(t.lanes, tap_e, p.he, m - p.he);
                for (int j = 0; j < 2; ++j)             // transposed: what the node takes from y_s, y_e
                    for (int c = 0; c < 4; ++c) {
                        const int i = s + 4 * k + c;
                        push(t.lanes, op != TILE_DT || i >= e ? 0.0 : (j ? tap(ce, bh[be], e, i) : tap(cs, bh[b], s, i)));
                    }
                // junctions inside: the node that is one, which of them it is, their taps, and
                // (transposed) what the nodes take from them
                int own = -1;
                for (int c = 0; c < 4; ++c) {
                    const int j = op == TILE_DT ? -1 : inside(4 * k + c);
                    if (j >= 0) own = j;
                    push(t.lanes_in, j >= 0 ? 1.0 : 0.0);
                }
                for (int j = 0; j < 4; ++j) push(t.lanes_in, j == own ? 1.0 : 0.0);
                for (int j = 0; j < kTileIn; ++j) {
                    if (j < ni) put_taps(t.lanes_in, tap_j[j], hi[j], sb[b + 1 + j] - s - hi[j]);
                    else for (int x = 0; x < 8; ++x) t.lanes_in.push_back(0.f);
                }
                for (int j = 0; j < kTileIn; ++j)
                    for (int c = 0; c < 4; ++c) {
                        const int i = s + 4 * k + c;
                        push(t.lanes_in, op != TILE_DT || i >= e || j >= ni
                                             ? 0.0
                                             : tap(&taps[(size_t)(b + 1 + j) * kTapW], bh[b + 1 + j], sb[b + 1 + j], i));
                    }
            }
        }
    }
    return std::string();
}

}  // namespace loss
