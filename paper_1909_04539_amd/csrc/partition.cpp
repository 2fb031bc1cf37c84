// Host side of the partitioned solve: block factors, spikes and the inverse
// of the interface system, all in FP64, computed once per shared matrix.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "factor_rows.h"
#include "internal.h"

namespace sbs {
namespace {

constexpr int kMaxBlocks = 64;
constexpr int kMaxInterface = 90;  // interface unknowns: the FP64 inverse stays under 64 KB of LDS

size_t align16(size_t v) { return (v + 15) / 16 * 16; }
size_t align256(size_t v) { return (v + 255) / 256 * 256; }  // each blob starts as a device allocation would

// Gauss-Jordan inverse with partial pivoting, in place (row-major n x n).  Row
// c of `a` is 0 before column c when it is used, and that of `inv` after the
// last column that a pivot has reached (`last`).
bool invert(std::vector<double> &a, int n) {
    std::vector<double> inv((size_t)n * n, 0.0);
    for (int i = 0; i < n; ++i) inv[(size_t)i * n + i] = 1.0;
    int last = 0;
    for (int c = 0; c < n; ++c) {
        int piv = c;
        for (int r = c + 1; r < n; ++r)
            if (std::fabs(a[(size_t)r * n + c]) > std::fabs(a[(size_t)piv * n + c])) piv = r;
        const double pv = a[(size_t)piv * n + c];
        if (!std::isfinite(pv) || std::fabs(pv) < 1e-300) return false;
        if (piv != c)
            for (int k = 0; k < n; ++k) {
                std::swap(a[(size_t)piv * n + k], a[(size_t)c * n + k]);
                std::swap(inv[(size_t)piv * n + k], inv[(size_t)c * n + k]);
            }
        last = std::max(last, piv);
        const double s = 1.0 / pv;
        double *ac = a.data() + (size_t)c * n, *ic = inv.data() + (size_t)c * n;
        for (int k = c; k < n; ++k) ac[k] *= s;
        for (int k = 0; k <= last; ++k) ic[k] *= s;
        for (int r = 0; r < n; ++r) {
            if (r == c) continue;
            double *ar = a.data() + (size_t)r * n, *ir = inv.data() + (size_t)r * n;
            const double f = ar[c];
            if (f == 0.0) continue;
            for (int k = c; k < n; ++k) ar[k] -= f * ac[k];
            for (int k = 0; k <= last; ++k) ir[k] -= f * ic[k];
        }
    }
    for (double v : inv)
        if (!std::isfinite(v)) return false;
    a.swap(inv);
    return true;
}

// A bandwidth's factorisation and its solve of NC columns at once (x is
// [n][NC]; each column is solved as solve_tri_rows / solve_penta_rows solve it.
// One column is a chain of dependent operations, several fill the time between
// them).
struct Tri {
    using Row = TriRow<double>;
    using Row32 = TriRow<float>;
    static constexpr int kind = SBS_TRI, h = 1;
    template <class Coef>
    static bool factor(int64_t n, Coef coef, Row *rows, int64_t *bad) {
        return factor_tri_rows(n, coef, rows, bad);
    }
    template <int NC>
    static void solve(int64_t n, const Row *r, double *x) {
        double y[NC] = {};
        for (int64_t i = 0; i < n; ++i)
            for (int c = 0; c < NC; ++c) y[c] = x[i * NC + c] = x[i * NC + c] * r[i].inv - r[i].a_s * y[c];
        for (int c = 0; c < NC; ++c) y[c] = 0.0;
        for (int64_t i = n - 1; i >= 0; --i)
            for (int c = 0; c < NC; ++c) y[c] = x[i * NC + c] = x[i * NC + c] - r[i].chat * y[c];
    }
};
struct Penta {
    using Row = PentaRow<double>;
    using Row32 = PentaRow<float>;
    static constexpr int kind = SBS_PENTA, h = 2;
    template <class Coef>
    static bool factor(int64_t n, Coef coef, Row *rows, int64_t *bad) {
        return factor_penta_rows(n, coef, rows, bad);
    }
    template <int NC>
    static void solve(int64_t n, const Row *r, double *x) {
        double y1[NC] = {}, y2[NC] = {};
        for (int64_t i = 0; i < n; ++i)
            for (int c = 0; c < NC; ++c) {
                const double g = x[i * NC + c] * r[i].inv - r[i].eps_s * y2[c] - r[i].beta_s * y1[c];
                x[i * NC + c] = g;
                y2[c] = y1[c];
                y1[c] = g;
            }
        for (int c = 0; c < NC; ++c) y1[c] = y2[c] = 0.0;
        for (int64_t i = n - 1; i >= 0; --i)
            for (int c = 0; c < NC; ++c) {
                const double v = x[i * NC + c] - r[i].gamma * y1[c] - r[i].delta * y2[c];
                x[i * NC + c] = v;
                y2[c] = y1[c];
                y1[c] = v;
            }
    }
};

struct HostPlan {
    int lb = 0, P = 0, Nr = 0, D = 0;
    std::vector<unsigned char> fac;  // D*lb FP64 rows (distinct blocks only)
    std::vector<double> spk;         // D*lb*2h
    std::vector<double> rinv;        // Nr*Nr
    std::vector<int> map;            // block p -> stored block map[p]
};

// Accuracy gate of a plan.  The partition reaches the same solution as the
// sweeps in exact arithmetic, but it rounds differently: through the block
// pivots and the interface inverse.  A block whose own pivots are tiny, or an
// ill-conditioned matrix whose interface system amplifies rounding, can move
// the partitioned result far from the recurrences of Sections 3.1 / 4.1 even
// when every pivot is nonzero.  So the plan is run on the host, in FP64, on a
// few seeded right-hand sides and compared with the sweep recurrences on the
// whole matrix; a plan whose result differs by more than kPlanTolerance
// (relative, per column, infinity norm) is dropped and the sweeps serve that
// matrix.  Four right-hand sides are uniform in every row; two are A x of a
// uniform x, as large in each row as its coefficients: with uniform ones the
// unknowns of small rows outweigh all others, and a plan that loses the
// unknowns of large rows would pass.  For those two the plan may be as near to
// that x instead (the periodic recurrences lose digits of their own where the
// first row is large).
constexpr double kPlanTolerance = 1e-13;
constexpr int kUniformChecks = 4, kChecks = 6;  // right-hand sides: uniform ones, all

using Columns = std::vector<double>;  // [n][kChecks]

// The right-hand sides of the gate, their solutions by the recurrences that
// the sweep kernels run, on the whole matrix (Section 3.3 for a periodic one:
// y = A'^{-1} d, then x = y - (wt.d) z), and the x that right-hand side q was
// formed from (q >= kUniformChecks); one of these serves every plan of a matrix.
struct Gate {
    Columns d, x, from;
};

template <class M>
Gate make_gate(bool periodic, int64_t n, const double *bands) {
    constexpr int h = M::h;
    // xorshift64, a fixed seed for each column (side by side, as the solves are)
    uint64_t st[kChecks];
    for (int q = 0; q < kChecks; ++q) st[q] = 0x9e3779b97f4a7c15ull * (2 * q + 1);
    Gate g;
    g.from.resize((size_t)n * kChecks);
    for (int64_t i = 0; i < n; ++i)
        for (int q = 0; q < kChecks; ++q) {
            st[q] ^= st[q] << 13;
            st[q] ^= st[q] >> 7;
            st[q] ^= st[q] << 17;
            // U[-1, 1): the top bits as the mantissa of a number in [2, 4)
            const uint64_t bits = 0x4000000000000000ull | st[q] >> 12;
            double u;
            std::memcpy(&u, &bits, 8);
            g.from[i * kChecks + q] = u - 3.0;
        }
    g.d = g.from;
    for (int64_t i = 0; i < n; ++i)
        for (int q = kUniformChecks; q < kChecks; ++q) {
            double ax = 0.0;
            for (int k = 0; k < 2 * h + 1; ++k) {
                int64_t col = i + k - h;
                if (periodic) col = col < 0 ? col + n : col >= n ? col - n : col;
                if (col >= 0 && col < n) ax += bands[(int64_t)k * n + i] * g.from[col * kChecks + q];
            }
            g.d[i * kChecks + q] = ax;
        }
    g.x = g.d;
    auto cf = [&](int k, int64_t i) -> double {
        const int64_t col = i + k - h;
        return !periodic && (col < 0 || col >= n) ? 0.0 : bands[(int64_t)k * n + i];
    };
    int64_t bad = -1;
    std::vector<typename M::Row> rows(n);
    if constexpr (M::kind == SBS_TRI)
        if (periodic) {
            std::vector<PeriodicRow<double>> r(n);
            if (!factor_periodic_rows(n, cf, r.data(), &bad)) return g;
            double acc[kChecks] = {};
            for (int64_t i = 0; i < n; ++i) {
                rows[i] = {r[i].a_s, r[i].chat, r[i].inv, 0.0};
                for (int q = 0; q < kChecks; ++q) acc[q] += r[i].wt * g.x[i * kChecks + q];
            }
            M::template solve<kChecks>(n, rows.data(), g.x.data());
            for (int64_t i = 0; i < n; ++i)
                for (int q = 0; q < kChecks; ++q) g.x[i * kChecks + q] -= acc[q] * r[i].z;
            return g;
        }
    if (M::factor(n, cf, rows.data(), &bad)) M::template solve<kChecks>(n, rows.data(), g.x.data());
    return g;
}

// Whether a plan's solutions (`plan`, in place) are the gate's; a NaN is not.
template <typename PlanSolve>
bool passes(const Gate &g, PlanSolve plan) {
    Columns b = g.d;
    plan(b);
    // largest entry of `a` and of b - a, column by column (a NaN in b makes sum one)
    double num[kChecks], den[kChecks], sum[kChecks];
    auto compare = [&](const Columns &a) {
        for (int q = 0; q < kChecks; ++q) num[q] = den[q] = sum[q] = 0.0;
        for (size_t i = 0; i < b.size(); i += kChecks)
            for (int q = 0; q < kChecks; ++q) {
                const double e = std::fabs(b[i + q] - a[i + q]), v = std::fabs(a[i + q]);
                num[q] = e > num[q] ? e : num[q];
                den[q] = v > den[q] ? v : den[q];
                sum[q] += b[i + q] * 0.0;
            }
    };
    auto agrees = [&](int q) { return num[q] <= kPlanTolerance * den[q] && sum[q] == 0.0; };
    compare(g.x);
    bool all = true, scaled = true;
    for (int q = 0; q < kChecks; ++q) (q < kUniformChecks ? all : scaled) &= agrees(q);
    if (!all || scaled) return all;
    compare(g.from);
    for (int q = kUniformChecks; q < kChecks; ++q) all &= agrees(q);
    return all;
}

// The plan's own solve of the gate's columns, as the kernel runs it: block
// solves, interface unknowns from the stored inverse, correction.
template <class M>
void plan_solve(const HostPlan &hp, bool periodic, int64_t n, Columns &x) {
    constexpr int h = M::h, C = kChecks;
    const int lb = hp.lb, P = hp.P, Nr = hp.Nr;
    const auto *fac = reinterpret_cast<const typename M::Row *>(hp.fac.data());
    std::vector<double> g((size_t)P * lb * C, 0.0), y((size_t)std::max(Nr, 1) * C, 0.0);
    std::copy(x.begin(), x.end(), g.begin());
    for (int p = 0; p < P; ++p)
        M::template solve<C>(lb, fac + (int64_t)hp.map[p] * lb, g.data() + (int64_t)p * lb * C);
    auto has_next = [&](int p) { return periodic || p <= P - 2; };
    auto has_prev = [&](int p) { return periodic || p >= 1; };
    auto prev = [&](int p) { return p == 0 ? P - 1 : p - 1; };
    for (int p = 0; p < P; ++p)
        for (int c = 0; c < h; ++c)
            for (int q = 0; q < C; ++q) {
                if (has_next(p)) y[(2 * h * p + c) * C + q] = g[((int64_t)p * lb + lb - h + c) * C + q];
                if (has_prev(p)) y[(2 * h * prev(p) + h + c) * C + q] = g[((int64_t)p * lb + c) * C + q];
            }
    for (int p = 0; p < P; ++p) {
        double xt[2][C] = {}, xb[2][C] = {};
        for (int c = 0; c < h; ++c) {
            if (has_next(p))
                for (int k = 0; k < Nr; ++k)
                    for (int q = 0; q < C; ++q)
                        xt[c][q] += hp.rinv[(size_t)(2 * h * p + h + c) * Nr + k] * y[(size_t)k * C + q];
            if (has_prev(p))
                for (int k = 0; k < Nr; ++k)
                    for (int q = 0; q < C; ++q)
                        xb[c][q] += hp.rinv[(size_t)(2 * h * prev(p) + c) * Nr + k] * y[(size_t)k * C + q];
        }
        const double *sp = hp.spk.data() + (size_t)hp.map[p] * lb * 2 * h;
        for (int t = 0; t < lb; ++t) {
            const int64_t i = (int64_t)p * lb + t;
            if (i >= n) break;
            for (int q = 0; q < C; ++q) {
                double v = g[i * C + q];
                for (int c = 0; c < h; ++c) v -= sp[t * 2 * h + c] * xt[c][q];
                for (int c = 0; c < h; ++c) v -= sp[t * 2 * h + h + c] * xb[c][q];
                x[i * C + q] = v;
            }
        }
    }
}

// `periodic` wraps a tridiagonal matrix
// round (row 0 couples to row n-1 and back), which needs n to be a whole
// number of blocks: then block 0's left neighbour is block P-1 and block
// P-1's right neighbour is block 0, and the interface system gains that pair.
template <class M>
bool build_plan(bool periodic, int64_t n, const double *bands, int lb, const Gate &gate, HostPlan &hp) {
    using Row = typename M::Row;
    constexpr int h = M::h;
    const int P = (int)((n + lb - 1) / lb);
    const int pairs = periodic ? P : P - 1;
    if (P > kMaxBlocks || lb < 2 * h || 2 * h * pairs > kMaxInterface) return false;
    if (periodic && (n % lb != 0 || P < 2)) return false;
    const int64_t npad = (int64_t)P * lb;
    std::vector<Row> rows(npad);
    std::vector<double> spk((size_t)npad * 2 * h, 0.0);
    // Coefficient k of global row i restricted to block p (identity past n).
    auto local = [&](int p, int k, int64_t i) -> double {
        if (i >= n) return k == h ? 1.0 : 0.0;
        const int64_t col = i + k - h;
        if (col < (int64_t)p * lb || col >= (int64_t)(p + 1) * lb || col >= n) return 0.0;
        return bands[(int64_t)k * n + i];
    };
    // Entry of row i < n in column col (any index; wrapped when periodic).
    auto entry = [&](int64_t i, int64_t col) -> double {
        if (i >= n) return 0.0;
        int64_t d = col - i;
        if (periodic) {
            d = ((d % n) + n) % n;
            if (d > n / 2) d -= n;
        } else if (col < 0 || col >= n) {
            return 0.0;
        }
        return (d >= -h && d <= h) ? bands[(int64_t)(d + h) * n + i] : 0.0;
    };
    for (int p = 0; p < P; ++p) {
        const int64_t r0 = (int64_t)p * lb;
        int64_t bad = -1;
        if (!M::factor(lb, [&](int k, int64_t t) { return local(p, k, r0 + t); }, rows.data() + r0, &bad)) return false;
        double *v = spk.data() + (size_t)r0 * 2 * h;
        for (int t = 0; t < lb; ++t)
            for (int c = 0; c < h; ++c) {
                // Right spike columns: coupling of row r0+t to column r0+lb+c
                // (block p+1's first unknowns; none past the last block unless periodic).
                if (p < P - 1 || periodic) v[t * 2 * h + c] = entry(r0 + t, r0 + lb + c);
                // Left spike columns: coupling of row r0+t to column r0-h+c.
                if (p > 0 || periodic) v[t * 2 * h + h + c] = entry(r0 + t, r0 - h + c);
            }
        M::template solve<2 * h>(lb, rows.data() + r0, v);
    }
    // Interface system.  Unknown order: pair q holds (bottom h of block q,
    // top h of block q+1), q = 0..P-2, and q = P-1 (block P-1, block 0) when
    // periodic.
    const int Nr = 2 * h * pairs;
    std::vector<double> R((size_t)Nr * Nr, 0.0);
    const auto next = [&](int p) { return p == P - 1 ? 0 : p + 1; };
    const auto prev = [&](int p) { return p == 0 ? P - 1 : p - 1; };
    const auto has_next = [&](int p) { return periodic || p <= P - 2; };
    const auto has_prev = [&](int p) { return periodic || p >= 1; };
    auto ibot = [&](int p, int c) { return 2 * h * p + c; };              // bottom of block p
    auto itop = [&](int p, int c) { return 2 * h * prev(p) + h + c; };    // top of block p
    auto V = [&](int p, int t, int c) { return spk[(size_t)((int64_t)p * lb + t) * 2 * h + c]; };
    auto Wt = [&](int p, int t, int c) { return spk[(size_t)((int64_t)p * lb + t) * 2 * h + h + c]; };
    for (int p = 0; p < P; ++p) {
        for (int c = 0; c < h; ++c) {
            // equation of block p's local row t, for its interface rows
            for (int side = 0; side < 2; ++side) {
                int row, t;
                if (side == 0) {  // bottom rows
                    if (!has_next(p)) continue;
                    row = ibot(p, c);
                    t = lb - h + c;
                } else {  // top rows
                    if (!has_prev(p)) continue;
                    row = itop(p, c);
                    t = c;
                }
                R[(size_t)row * Nr + row] += 1.0;
                for (int c2 = 0; c2 < h; ++c2) {
                    if (has_next(p)) R[(size_t)row * Nr + itop(next(p), c2)] += V(p, t, c2);
                    if (has_prev(p)) R[(size_t)row * Nr + ibot(prev(p), c2)] += Wt(p, t, c2);
                }
            }
        }
    }
    if (Nr > 0 && !invert(R, Nr)) return false;
    hp.lb = lb;
    hp.P = P;
    hp.Nr = Nr;
    // Blocks whose factor rows and spikes are bit-identical (every interior
    // block of a matrix with constant bands) are stored once.
    const size_t rb = sizeof(Row) * lb, sb = sizeof(double) * lb * 2 * h;
    hp.map.assign(P, -1);
    hp.fac.clear();
    hp.spk.clear();
    for (int p = 0; p < P; ++p) {
        const unsigned char *rp = reinterpret_cast<const unsigned char *>(rows.data() + (int64_t)p * lb);
        const double *sp = spk.data() + (size_t)p * lb * 2 * h;
        for (int q = 0; q < hp.D && hp.map[p] < 0; ++q)
            if (!std::memcmp(hp.fac.data() + q * rb, rp, rb) && !std::memcmp(hp.spk.data() + q * lb * 2 * h, sp, sb))
                hp.map[p] = q;
        if (hp.map[p] < 0) {
            hp.map[p] = hp.D++;
            hp.fac.insert(hp.fac.end(), rp, rp + rb);
            hp.spk.insert(hp.spk.end(), sp, sp + (size_t)lb * 2 * h);
        }
    }
    hp.rinv.swap(R);
    return passes(gate, [&](Columns &x) { plan_solve<M>(hp, periodic, n, x); });
}

// ---------------------------------------------------------------------------
// Separator partition (SepPlan).

constexpr int kMaxSepInterface = 128;  // separator unknowns: the FP64 inverse stays within 128 KB of LDS

struct SepHostPlan {
    int lb = 0, P = 0, Nr = 0, D = 0;
    std::vector<unsigned char> fac;  // D*lb FP64 rows
    std::vector<double> spk;         // D*lb*2h: V (own separator), W (previous separator)
    std::vector<double> scf;         // D*h*(2h+1)
    std::vector<double> sinv;        // Nr*Nr
    std::vector<int> map;
    int kofs = 0, kw = 0;            // window of the S^{-1} product (sep_window)
};

// Entries of S^{-1} that cannot matter, and the window of columns the
// kernel's product then reads.  The separators of blocks far apart are
// coupled only through the spikes, which decay row by row for a diagonally
// dominant or positive definite matrix, so most of S^{-1} is far below its
// row's largest entry (for the 1024-row hyperdiffusion matrix in 32-row
// blocks, entries two separators apart are below 1e-24 of it).  An entry
// S^{-1}_ij is set to 0 if both its magnitude and |S^{-1}_ij| s_j, with s_j the
// largest entry of row j of S, are at most 2^-60 / Nr of the largest in its
// row.  A separator right-hand side yhat = S z is as large as its row of S
// makes it (|yhat_j| <= Nr s_j max |z|), and S^{-1}_ij as small, so it is the
// weighted entry that tells whether z_i depends on it; the entry itself bounds
// the dropped part of any z_i = sum_j S^{-1}_ij yhat_j by
// 2^-60 max_j |S^{-1}_ij| max |yhat|, below 1 / (128 Nr) of the rounding
// error bound of the product itself.  The product is done in 16-row tiles of
// S^{-1}; tile t (rows 16t .. 16t + 15) reads columns k0 .. k0 + kw - 1 with
// k0 = min(max(16t + kofs, 0), max(Nr4 - kw, 0)), Nr4 = Nr rounded up to 4,
// which holds every nonzero entry of the tile's rows.  kw = 0: every column.
// scale: the s_j.
void sep_window(std::vector<double> &S, const std::vector<double> &scale, int Nr, int &kofs, int &kw) {
    kofs = kw = 0;
    if (Nr <= 0) return;
    for (int i = 0; i < Nr; ++i) {
        double *row = S.data() + (size_t)i * Nr;
        double mx = 0.0, mxs = 0.0;
        for (int j = 0; j < Nr; ++j) {
            mx = std::max(mx, std::fabs(row[j]));
            mxs = std::max(mxs, std::fabs(row[j]) * scale[j]);
        }
        const double thr = std::ldexp(mx, -60) / Nr, thrs = std::ldexp(mxs, -60) / Nr;
        for (int j = 0; j < Nr; ++j)
            if (std::fabs(row[j]) <= thr && std::fabs(row[j]) * scale[j] <= thrs) row[j] = 0.0;
    }
    const int mt = (Nr + 15) / 16, Nr4 = (Nr + 3) / 4 * 4;
    std::vector<int> lo(mt, Nr), hi(mt, -1);
    for (int i = 0; i < Nr; ++i)
        for (int j = 0; j < Nr; ++j)
            if (S[(size_t)i * Nr + j] != 0.0) {
                lo[i / 16] = std::min(lo[i / 16], j);
                hi[i / 16] = std::max(hi[i / 16], j);
            }
    int ofs = 0;
    for (int t = 0; t < mt; ++t) ofs = std::min(ofs, lo[t] - 16 * t);
    ofs = -((-ofs + 3) / 4 * 4);
    for (int w = 4; w < Nr4; w += 4) {
        bool holds = true;
        for (int t = 0; t < mt && holds; ++t) {
            const int k0 = std::min(std::max(16 * t + ofs, 0), std::max(Nr4 - w, 0));
            holds = lo[t] >= k0 && hi[t] < k0 + w;
        }
        if (holds) {
            kofs = ofs;
            kw = w;
            return;
        }
    }
}

// The separator plan's own solve of the gate's columns (x: [n][kChecks]), as
// the kernel runs it: block sweeps (separator rows pass through unchanged),
// separator right-hand sides yhat, separators z = S^{-1} yhat, interior
// correction.
template <class M>
void sep_plan_solve(const SepHostPlan &hp, bool periodic, int64_t n, double *x) {
    constexpr int h = M::h, nb = 2 * h + 1, C = kChecks;
    const int lb = hp.lb, P = hp.P, Nr = hp.Nr;
    const auto *fac = reinterpret_cast<const typename M::Row *>(hp.fac.data());
    auto has_sep = [&](int p) { return periodic || p < P - 1; };
    auto has_prev = [&](int p) { return periodic || p >= 1; };
    auto prev = [&](int p) { return p == 0 ? P - 1 : p - 1; };
    auto next = [&](int p) { return p == P - 1 ? 0 : p + 1; };
    std::vector<double> g((size_t)P * lb * C, 0.0), yh((size_t)std::max(Nr, 1) * C, 0.0), z = yh;
    std::copy(x, x + n * C, g.begin());
    for (int p = 0; p < P; ++p)
        M::template solve<C>(lb, fac + (int64_t)hp.map[p] * lb, g.data() + (int64_t)p * lb * C);
    for (int p = 0; p < P; ++p) {
        if (!has_sep(p)) continue;
        const double *cf = hp.scf.data() + (size_t)hp.map[p] * h * nb;
        for (int c = 0; c < h; ++c) {
            double *y = yh.data() + (size_t)(h * p + c) * C;
            for (int q = 0; q < C; ++q) y[q] = x[((int64_t)p * lb + lb - h + c) * C + q];
            for (int d = 0; d < nb; ++d) {
                const int t = lb - h + c + d - h;  // column, relative to the block's first row
                if (t >= lb - h && t < lb) continue;
                const double *v = g.data() + (t < lb ? (int64_t)p * lb + t : (int64_t)next(p) * lb + t - lb) * C;
                for (int q = 0; q < C; ++q) y[q] -= cf[c * nb + d] * v[q];
            }
        }
    }
    for (int r = 0; r < Nr; ++r)
        for (int k = 0; k < Nr; ++k)
            for (int q = 0; q < C; ++q) z[(size_t)r * C + q] += hp.sinv[(size_t)r * Nr + k] * yh[(size_t)k * C + q];
    for (int p = 0; p < P; ++p) {
        const double *sp = hp.spk.data() + (size_t)hp.map[p] * lb * 2 * h;
        for (int t = 0; t < lb; ++t) {
            const int64_t i = (int64_t)p * lb + t;
            if (i >= n) break;
            const bool sep = has_sep(p) && t >= lb - h;
            for (int q = 0; q < C; ++q) {
                double v = sep ? z[(size_t)(h * p + t - (lb - h)) * C + q] : g[i * C + q];
                for (int c = 0; c < h && !sep; ++c) {
                    if (has_sep(p)) v -= sp[t * 2 * h + c] * z[(size_t)(h * p + c) * C + q];
                    if (has_prev(p)) v -= sp[t * 2 * h + h + c] * z[(size_t)(h * prev(p) + c) * C + q];
                }
                x[i * C + q] = v;
            }
        }
    }
}

// `periodic` wraps a tridiagonal matrix round (needs n a whole
// number P >= 2 of blocks; every block then has a separator).  gate: the
// accuracy gate (null: the caller checks the whole).
template <class M>
bool build_sep_plan(bool periodic, int64_t n, const double *bands, int lb, const Gate *gate, SepHostPlan &hp) {
    using Row = typename M::Row;
    constexpr int h = M::h, nb = 2 * h + 1;
    const int P = (int)((n + lb - 1) / lb);
    if (periodic && (n % lb != 0 || P < 2)) return false;
    const int nsep = periodic ? P : P - 1;
    if (P > kMaxBlocks || lb < 2 * h + 1 || h * nsep > kMaxSepInterface) return false;
    const int64_t npad = (int64_t)P * lb;
    auto has_sep = [&](int p) { return periodic || p < P - 1; };
    auto has_prev = [&](int p) { return periodic || p >= 1; };
    auto prev = [&](int p) { return p == 0 ? P - 1 : p - 1; };
    auto next = [&](int p) { return p == P - 1 ? 0 : p + 1; };
    auto interior = [&](int p) { return has_sep(p) ? lb - h : lb; };
    // Entry of row i < n in column col (any index; wrapped when periodic).
    auto entry = [&](int64_t i, int64_t col) -> double {
        if (i >= n) return 0.0;
        int64_t d = col - i;
        if (periodic) {
            d = ((d % n) + n) % n;
            if (d > n / 2) d -= n;
        } else if (col < 0 || col >= n) {
            return 0.0;
        }
        return (d >= -h && d <= h) ? bands[(int64_t)(d + h) * n + i] : 0.0;
    };
    std::vector<Row> rows(npad);
    std::vector<double> spk((size_t)npad * 2 * h, 0.0), scf((size_t)P * h * nb, 0.0);
    for (int p = 0; p < P; ++p) {
        const int64_t r0 = (int64_t)p * lb;
        const int ni = interior(p);
        // the interior block: coefficients among its own interior columns,
        // identity on separator rows and past the end
        auto local = [&](int k, int64_t t) -> double {
            const int64_t i = r0 + t;
            if (i >= n || t >= ni) return k == h ? 1.0 : 0.0;
            const int64_t ct = t + k - h;
            if (ct < 0 || ct >= ni || r0 + ct >= n) return 0.0;
            return bands[(int64_t)k * n + i];
        };
        int64_t bad = -1;
        if (!M::factor(lb, local, rows.data() + r0, &bad)) return false;
        double *v = spk.data() + (size_t)r0 * 2 * h;
        for (int t = 0; t < ni; ++t)
            for (int c = 0; c < h; ++c) {
                // V: the block's own separator rows r0 + ni + c
                if (has_sep(p)) v[t * 2 * h + c] = entry(r0 + t, r0 + ni + c);
                // W: the previous separator, rows r0 - h + c (wrapped for block 0)
                if (has_prev(p)) v[t * 2 * h + h + c] = entry(r0 + t, p == 0 ? n - h + c : r0 - h + c);
            }
        M::template solve<2 * h>(lb, rows.data() + r0, v);
        std::fill(v + ni * 2 * h, v + lb * 2 * h, 0.0);
        if (!has_sep(p)) continue;
        // band rows of the separator rows, without the separator columns
        for (int c = 0; c < h; ++c)
            for (int d = 0; d < nb; ++d) {
                const int t = ni + c + d - h;
                if (t >= ni && t < lb) continue;
                scf[((size_t)p * h + c) * nb + d] = entry(r0 + ni + c, r0 + t);
            }
    }
    // S: separator s (of block s), row c.  Unknown order h * s + c.
    const int Nr = h * nsep;
    std::vector<double> S((size_t)Nr * Nr, 0.0);
    auto V = [&](int p, int t, int c) { return spk[(size_t)((int64_t)p * lb + t) * 2 * h + c]; };
    auto W = [&](int p, int t, int c) { return spk[(size_t)((int64_t)p * lb + t) * 2 * h + h + c]; };
    for (int s = 0; s < nsep; ++s) {
        const int64_t r0 = (int64_t)s * lb;
        const int ni = lb - h, nx = next(s);
        for (int c = 0; c < h; ++c) {
            const int row = h * s + c;
            for (int c2 = 0; c2 < h; ++c2) S[(size_t)row * Nr + h * s + c2] += entry(r0 + ni + c, r0 + ni + c2);
            for (int d = 0; d < nb; ++d) {
                const int t = ni + c + d - h;
                const double cf = scf[((size_t)s * h + c) * nb + d];
                if (cf == 0.0) continue;
                if (t < ni) {  // interior row t of block s
                    for (int c2 = 0; c2 < h; ++c2) {
                        S[(size_t)row * Nr + h * s + c2] -= cf * V(s, t, c2);
                        if (has_prev(s)) S[(size_t)row * Nr + h * prev(s) + c2] -= cf * W(s, t, c2);
                    }
                } else {  // interior row t - lb of the next block
                    const int u = t - lb;
                    for (int c2 = 0; c2 < h; ++c2) {
                        S[(size_t)row * Nr + h * s + c2] -= cf * W(nx, u, c2);
                        if (has_sep(nx)) S[(size_t)row * Nr + h * nx + c2] -= cf * V(nx, u, c2);
                    }
                }
            }
        }
    }
    std::vector<double> scale(Nr, 0.0);
    for (int r = 0; r < Nr; ++r)
        for (int k = 0; k < Nr; ++k) scale[r] = std::max(scale[r], std::fabs(S[(size_t)r * Nr + k]));
    // rows of about the same size, by powers of two: the pivots chosen and every
    // rounding are then the same however the matrix's rows are scaled
    std::vector<double> two(Nr, 1.0);
    for (int r = 0; r < Nr; ++r) {
        if (!(scale[r] > 1e-300 && scale[r] < 1e300)) return false;
        two[r] = std::ldexp(1.0, -std::ilogb(scale[r]));
        for (int k = 0; k < Nr; ++k) S[(size_t)r * Nr + k] *= two[r];
    }
    if (Nr > 0 && !invert(S, Nr)) return false;
    for (int r = 0; r < Nr; ++r)
        for (int k = 0; k < Nr; ++k) S[(size_t)r * Nr + k] *= two[k];
    sep_window(S, scale, Nr, hp.kofs, hp.kw);
    hp.lb = lb;
    hp.P = P;
    hp.Nr = Nr;
    hp.D = 0;
    const size_t rb = sizeof(Row) * lb, sb = sizeof(double) * lb * 2 * h, cb = sizeof(double) * h * nb;
    hp.map.assign(P, -1);
    hp.fac.clear();
    hp.spk.clear();
    hp.scf.clear();
    for (int p = 0; p < P; ++p) {
        const unsigned char *rp = reinterpret_cast<const unsigned char *>(rows.data() + (int64_t)p * lb);
        const double *sp = spk.data() + (size_t)p * lb * 2 * h;
        const double *cp = scf.data() + (size_t)p * h * nb;
        for (int q = 0; q < hp.D && hp.map[p] < 0; ++q)
            if (!std::memcmp(hp.fac.data() + q * rb, rp, rb) && !std::memcmp(hp.spk.data() + q * lb * 2 * h, sp, sb) &&
                !std::memcmp(hp.scf.data() + (size_t)q * h * nb, cp, cb))
                hp.map[p] = q;
        if (hp.map[p] < 0) {
            hp.map[p] = hp.D++;
            hp.fac.insert(hp.fac.end(), rp, rp + rb);
            hp.spk.insert(hp.spk.end(), sp, sp + (size_t)lb * 2 * h);
            hp.scf.insert(hp.scf.end(), cp, cp + (size_t)h * nb);
        }
    }
    hp.sinv.swap(S);
    return !gate || passes(*gate, [&](Columns &x) { sep_plan_solve<M>(hp, periodic, n, x.data()); });
}

template <typename Row32, typename Row64>
Row32 narrow_row(const Row64 &r);
template <>
TriRow<float> narrow_row(const TriRow<double> &r) {
    return {(float)r.a_s, (float)r.chat, (float)r.inv, 0.0f};
}
template <>
PentaRow<float> narrow_row(const PentaRow<double> &r) {
    return {(float)r.eps_s, (float)r.beta_s, (float)r.inv, (float)r.gamma, (float)r.delta, 0.f, 0.f, 0.f};
}

// memcpy that accepts an empty source (an empty vector's data() may be null).
void copy_bytes(void *dst, const void *src, size_t bytes) {
    if (bytes) std::memcpy(dst, src, bytes);
}

// Serialise one plan as [fac | spk | rinv | map] in FP64 and in FP32.
template <typename Row64, typename Row32>
void serialise(const HostPlan &hp, std::vector<unsigned char> &b64, std::vector<unsigned char> &b32, PartPlan &pp) {
    const size_t nrow = hp.fac.size() / sizeof(Row64);
    const size_t map_bytes = align16(hp.map.size() * sizeof(int));
    pp.fac_bytes64 = align16(hp.fac.size());
    pp.spk_bytes64 = align16(hp.spk.size() * 8);
    pp.rinv_bytes64 = align16(hp.rinv.size() * 8);
    b64.assign(pp.fac_bytes64 + pp.spk_bytes64 + pp.rinv_bytes64 + map_bytes, 0);
    copy_bytes(b64.data(), hp.fac.data(), hp.fac.size());
    copy_bytes(b64.data() + pp.fac_bytes64, hp.spk.data(), hp.spk.size() * 8);
    copy_bytes(b64.data() + pp.fac_bytes64 + pp.spk_bytes64, hp.rinv.data(), hp.rinv.size() * 8);
    copy_bytes(b64.data() + pp.fac_bytes64 + pp.spk_bytes64 + pp.rinv_bytes64, hp.map.data(),
                hp.map.size() * sizeof(int));
    pp.fac_bytes32 = align16(nrow * sizeof(Row32));
    pp.spk_bytes32 = align16(hp.spk.size() * 4);
    pp.rinv_bytes32 = align16(hp.rinv.size() * 4);
    b32.assign(pp.fac_bytes32 + pp.spk_bytes32 + pp.rinv_bytes32 + map_bytes, 0);
    const Row64 *r64 = reinterpret_cast<const Row64 *>(hp.fac.data());
    Row32 *r32 = reinterpret_cast<Row32 *>(b32.data());
    for (size_t i = 0; i < nrow; ++i) r32[i] = narrow_row<Row32>(r64[i]);
    float *s32 = reinterpret_cast<float *>(b32.data() + pp.fac_bytes32);
    for (size_t i = 0; i < hp.spk.size(); ++i) s32[i] = (float)hp.spk[i];
    float *q32 = reinterpret_cast<float *>(b32.data() + pp.fac_bytes32 + pp.spk_bytes32);
    for (size_t i = 0; i < hp.rinv.size(); ++i) q32[i] = (float)hp.rinv[i];
    copy_bytes(b32.data() + pp.fac_bytes32 + pp.spk_bytes32 + pp.rinv_bytes32, hp.map.data(),
                hp.map.size() * sizeof(int));
    pp.map_bytes = map_bytes;
    pp.D = hp.D;
}

// Serialise one separator plan as [fac | spk | scf | sinv | map] in FP64 and FP32.
template <typename Row64, typename Row32>
void serialise_sep(const SepHostPlan &hp, std::vector<unsigned char> &b64, std::vector<unsigned char> &b32,
                   SepPlan &pp) {
    const size_t nrow = hp.fac.size() / sizeof(Row64);
    const size_t map_bytes = align16(hp.map.size() * sizeof(int));
    pp.fac_bytes64 = align16(hp.fac.size());
    pp.spk_bytes64 = align16(hp.spk.size() * 8);
    pp.scf_bytes64 = align16(hp.scf.size() * 8);
    pp.sinv_bytes64 = align16(hp.sinv.size() * 8);
    b64.assign(pp.fac_bytes64 + pp.spk_bytes64 + pp.scf_bytes64 + pp.sinv_bytes64 + map_bytes, 0);
    unsigned char *at = b64.data();
    copy_bytes(at, hp.fac.data(), hp.fac.size());
    copy_bytes(at += pp.fac_bytes64, hp.spk.data(), hp.spk.size() * 8);
    copy_bytes(at += pp.spk_bytes64, hp.scf.data(), hp.scf.size() * 8);
    copy_bytes(at += pp.scf_bytes64, hp.sinv.data(), hp.sinv.size() * 8);
    copy_bytes(at += pp.sinv_bytes64, hp.map.data(), hp.map.size() * sizeof(int));
    pp.fac_bytes32 = align16(nrow * sizeof(Row32));
    pp.spk_bytes32 = align16(hp.spk.size() * 4);
    pp.scf_bytes32 = align16(hp.scf.size() * 4);
    pp.sinv_bytes32 = align16(hp.sinv.size() * 4);
    b32.assign(pp.fac_bytes32 + pp.spk_bytes32 + pp.scf_bytes32 + pp.sinv_bytes32 + map_bytes, 0);
    const Row64 *r64 = reinterpret_cast<const Row64 *>(hp.fac.data());
    Row32 *r32 = reinterpret_cast<Row32 *>(b32.data());
    for (size_t i = 0; i < nrow; ++i) r32[i] = narrow_row<Row32>(r64[i]);
    auto put = [](unsigned char *dst, const std::vector<double> &src) {
        float *f = reinterpret_cast<float *>(dst);
        for (size_t i = 0; i < src.size(); ++i) f[i] = (float)src[i];
    };
    unsigned char *q = b32.data() + pp.fac_bytes32;
    put(q, hp.spk);
    put(q += pp.spk_bytes32, hp.scf);
    put(q += pp.scf_bytes32, hp.sinv);
    copy_bytes(q += pp.sinv_bytes32, hp.map.data(), hp.map.size() * sizeof(int));
    pp.map_bytes = map_bytes;
    pp.D = hp.D;
    pp.lb = hp.lb;
    pp.P = hp.P;
    pp.Nr = hp.Nr;
    pp.kofs = hp.kofs;
    pp.kw = hp.kw;
}

// The one-wave-per-block mixed-precision kernel's copy of a separator plan:
// each pass's coefficients contiguous, so that a wave reads a run of rows
// with a few wide scalar loads.  Per distinct block (FP32, from the plan):
// forward coefficients (tri a/den, 1/den; penta eps/alpha, beta/alpha,
// 1/alpha), backward coefficients (tri chat; penta gamma, delta), spikes;
// per block (FP64): the original band rows, 0 outside the matrix; and S^{-1}
// (FP32) with its rows padded with zeros to a multiple of 8 entries.
template <typename Row32>
void serialise_refine(const SepHostPlan &hp, const std::vector<unsigned char> &b32, const SepPlan &sp, int kind,
                      int64_t n, const double *bands, std::vector<unsigned char> &out, RefinePlan &rp) {
    const int h = kind / 2, nb = 2 * h + 1, lb = hp.lb, D = hp.D, P = hp.P;
    const int F = kind == SBS_TRI ? 2 : 3, Bk = kind == SBS_TRI ? 1 : 2;
    rp.fwd = 0;
    rp.bwd = align256(rp.fwd + (size_t)D * lb * F * 4);
    rp.spk = align256(rp.bwd + (size_t)D * lb * Bk * 4);
    rp.band = align256(rp.spk + (size_t)D * lb * 2 * h * 4);
    rp.ldsinv = (hp.Nr + 7) / 8 * 8;
    rp.sinv = align256(rp.band + (size_t)P * lb * nb * 8);
    const size_t total = align256(rp.sinv + (size_t)hp.Nr * rp.ldsinv * 4);
    out.assign(total, 0);
    const Row32 *rows = reinterpret_cast<const Row32 *>(b32.data());
    float *fwd = reinterpret_cast<float *>(out.data() + rp.fwd);
    float *bwd = reinterpret_cast<float *>(out.data() + rp.bwd);
    for (size_t i = 0; i < (size_t)D * lb; ++i) {
        if constexpr (sizeof(Row32) == sizeof(TriRow<float>)) {
            fwd[2 * i] = rows[i].a_s;
            fwd[2 * i + 1] = rows[i].inv;
            bwd[i] = rows[i].chat;
        } else {
            fwd[3 * i] = rows[i].eps_s;
            fwd[3 * i + 1] = rows[i].beta_s;
            fwd[3 * i + 2] = rows[i].inv;
            bwd[2 * i] = rows[i].gamma;
            bwd[2 * i + 1] = rows[i].delta;
        }
    }
    copy_bytes(out.data() + rp.spk, b32.data() + sp.fac_bytes32, (size_t)D * lb * 2 * h * 4);
    double *band = reinterpret_cast<double *>(out.data() + rp.band);
    for (int64_t i = 0; i < std::min<int64_t>(n, (int64_t)P * lb); ++i)
        for (int k = 0; k < nb; ++k) {
            const int64_t col = i + k - h;
            band[i * nb + k] = (col >= 0 && col < n) ? bands[(int64_t)k * n + i] : 0.0;
        }
    float *sinv = reinterpret_cast<float *>(out.data() + rp.sinv);
    for (int r = 0; r < hp.Nr; ++r)
        for (int k = 0; k < hp.Nr; ++k) sinv[(size_t)r * rp.ldsinv + k] = (float)hp.sinv[(size_t)r * hp.Nr + k];
}

// ---------------------------------------------------------------------------
// Segments (RefSeg) of a matrix that the one-wave-per-block mixed-precision
// kernels solve run of rows by run of rows.

struct HostSeg {
    int64_t lo = 0, hi = 0, a = 0, b = 0;  // rows solved, rows of the result
    int same = -1;                         // an earlier segment with the same rows (constant bands), or -1
    SepHostPlan hp;
    SepPlan sp;                            // blob sizes and RefinePlan offsets
    std::vector<unsigned char> b32, rec;   // serialised plan, the kernel's copy
};

// The bands of rows lo .. hi - 1 as a matrix of their own (couplings to rows
// outside dropped).
std::vector<double> sub_bands(int kind, int64_t n, const double *bands, int64_t lo, int64_t hi) {
    const int h = kind / 2;
    const int64_t ns = hi - lo;
    std::vector<double> out((size_t)kind * ns, 0.0);
    for (int k = 0; k < kind; ++k)
        for (int64_t i = 0; i < ns; ++i) {
            const int64_t col = i + k - h;
            if (col >= 0 && col < ns) out[(size_t)k * ns + i] = bands[(int64_t)k * n + lo + i];
        }
    return out;
}

// Whether what lies beyond the segment's cuts cannot matter for its result:
// with x_out the exact values just outside a cut, the truncated solution is
// off by A_seg^{-1} (coupling) x_out; every entry of A_seg^{-1} (coupling) on
// the result's rows has to be at most kSegDrop (2^-60: at most 2 h 2^-60 of
// the system's largest value in all, 1/32 of an FP64 rounding).
template <class M>
bool seg_independent(int64_t n, const double *bands, const HostSeg &s, const std::vector<double> &sub) {
    constexpr int h = M::h;
    const int64_t ns = s.hi - s.lo;
    std::vector<typename M::Row> rows(ns);
    int64_t bad = -1;
    if (!M::factor(ns, [&](int k, int64_t i) { return sub[(size_t)k * ns + i]; }, rows.data(), &bad)) return false;
    std::vector<double> v((size_t)ns * 2 * h, 0.0);
    for (int c = 0; c < h; ++c) {
        if (s.lo > 0)  // column lo - h + c meets rows lo .. lo + c
            for (int t = 0; t <= c; ++t) v[t * 2 * h + c] = bands[(int64_t)(c - t) * n + s.lo + t];
        if (s.hi < n)  // column hi + c meets rows hi - h + c .. hi - 1
            for (int t = c; t < h; ++t)
                v[(ns - h + t) * 2 * h + h + c] = bands[(int64_t)(2 * h + c - t) * n + s.hi - h + t];
    }
    M::template solve<2 * h>(ns, rows.data(), v.data());
    for (int64_t i = (s.a - s.lo) * 2 * h; i < (s.b - s.lo) * 2 * h; ++i)
        if (!(std::fabs(v[i]) <= kSegDrop)) return false;
    return true;
}

bool pays(int kind, int64_t shorter, int64_t longer, bool small) {
    return longer > 9 && shorter * 100 <= longer * (small ? 175 : kind == SBS_PENTA ? 140 : 145);
}

// The fewest equal runs of rows that fit blocks of `cap` rows with `halo` rows
// on either side: their number, and the 32-row blocks of all of them.
struct SegLayout {
    int64_t ns = 0, blocks = 0;
};
SegLayout seg_layout(int64_t n, int64_t cap, int64_t halo) {
    SegLayout l;
    if (n <= cap) return {1, (n + kSegLb - 1) / kSegLb};
    const int64_t core = cap - 2 * halo;
    l.ns = n <= 2 * (cap - halo) ? 2 : (n + core - 1) / core;
    const int64_t run = (n + l.ns - 1) / l.ns;
    for (int64_t k = 0; k < l.ns; ++k) {
        const int64_t lo = std::max<int64_t>(0, run * k - halo), hi = std::min(n, run * (k + 1) + halo);
        l.blocks += (std::max<int64_t>(hi - lo, 0) + kSegLb - 1) / kSegLb;
    }
    return l;
}

// Cuts the matrix into overlapping segments with the shortest halo that makes
// them independent; empty if there is none, or if the matrix is better solved
// whole.  Segments of seg_half blocks run two workgroups per CU, one of which
// computes while the other loads and stores, at about 36 us a block and 512K
// systems (pentadiagonal 49), one workgroup of twice the blocks at 55 (70 to
// 80): short ones unless their halos make 1.45 (1.4) times the blocks.  Batches
// that do not fill the GPU (32 systems a CU) take them up to 1.75 times, since
// they spread the rows over more CUs (n = 512, m = 1000: tridiagonal 19 -> 11
// us, pentadiagonal 27 -> 14; n = 480, m = 8000 20 and 18, m = 12876 30 and 34;
// m = 64000 115 and 122, 160 and 170).
// (256M unknowns, tridiagonal with 32-row halos n = 512 869 -> 805 us, n = 600
// 916 -> 827, n = 1500 951 -> 772; with 48-row ones n = 400 927 -> 711, n = 512
// would go from 869 to 909; pentadiagonal n = 300 1223 -> 1130, n = 1500
// 1436 -> 1352, n = 600 would go from 1295 to 1402, and nine whole blocks,
// n = 257, from 1123 to 1261.  Near 1.4 the two are close: n = 512 with random
// bands, halos of 32 or 40 rows, 22 blocks in three segments for 16, m = 400000
// 672 -> 637 us, m = 1M 1700 -> 1660.)
template <class M>
std::vector<HostSeg> build_segments(int64_t n, const double *bands, const Gate &gate) {
    constexpr int kind = M::kind;
    const int64_t most = (int64_t)seg_max_blocks(kind) * kSegLb, least = (int64_t)seg_half(kind) * kSegLb;
    // blocks of the whole matrix where one workgroup can hold it
    const int64_t whole = n <= kMaxWhole ? (n + kSegLb - 1) / kSegLb : 0;
    for (int halo = 8; halo <= kMaxHalo; halo += 8) {
        const SegLayout shorter = seg_layout(n, least, halo), longer = seg_layout(n, most, halo);
        const bool halves = shorter.ns <= kMaxSegs && pays(kind, shorter.blocks, whole ? whole : longer.blocks, whole > 0);
        const int64_t ns = halves ? shorter.ns : longer.ns;
        if (ns == 1 || ns > kMaxSegs) return {};
        std::vector<HostSeg> segs((size_t)ns);
        std::vector<std::vector<double>> sub((size_t)ns);
        bool ok = true;
        for (int64_t k = 0; k < ns && ok; ++k) {
            HostSeg &s = segs[k];
            // equal result runs (the last one shorter): with constant bands
            // every interior segment is the same matrix
            const int64_t run = (n + ns - 1) / ns;
            s.a = run * k;
            s.b = std::min<int64_t>(n, s.a + run);
            s.lo = std::max<int64_t>(0, s.a - halo);
            s.hi = std::min<int64_t>(n, s.b + halo);
            sub[k] = sub_bands(kind, n, bands, s.lo, s.hi);
            // an earlier segment with the same rows, couplings and place of
            // its result has answered already
            for (int64_t q = 0; q < k && s.same < 0; ++q) {
                const HostSeg &o = segs[q];
                if (o.same >= 0 || o.a - o.lo != s.a - s.lo || o.b - o.lo != s.b - s.lo || sub[q] != sub[k]) continue;
                bool alike = true;
                for (int64_t t = 0; t < kind / 2 && alike; ++t)
                    for (int b = 0; b < kind && alike; ++b)
                        alike = bands[b * n + s.lo + t] == bands[b * n + o.lo + t] &&
                                bands[b * n + s.hi - 1 - t] == bands[b * n + o.hi - 1 - t];
                if (alike && (o.lo > 0) == (s.lo > 0) && (o.hi < n) == (s.hi < n)) s.same = (int)q;
            }
            if (s.same < 0) ok = seg_independent<M>(n, bands, s, sub[k]);
        }
        if (!ok) continue;
        for (int64_t k = 0; k < ns; ++k) {
            HostSeg &s = segs[k];
            if (s.same >= 0) continue;
            if (!build_sep_plan<M>(false, s.hi - s.lo, sub[k].data(), kSegLb, nullptr, s.hp)) {
                ok = false;
                break;
            }
            std::vector<unsigned char> b64;
            serialise_sep<typename M::Row, typename M::Row32>(s.hp, b64, s.b32, s.sp);
            serialise_refine<typename M::Row32>(s.hp, s.b32, s.sp, kind, s.hi - s.lo, sub[k].data(), s.rec, s.sp.refine);
        }
        // the whole matrix's right-hand sides and solutions, segment by segment
        ok = ok && passes(gate, [&](Columns &x) {
            Columns f;
            for (const HostSeg &s : segs) {
                f.assign(gate.d.begin() + s.lo * kChecks, gate.d.begin() + s.hi * kChecks);
                sep_plan_solve<M>(s.same >= 0 ? segs[s.same].hp : s.hp, false, s.hi - s.lo, f.data());
                std::copy(f.begin() + (s.a - s.lo) * kChecks, f.begin() + (s.b - s.lo) * kChecks,
                          x.begin() + s.a * kChecks);
            }
        });
        if (!ok) continue;
        return segs;
    }
    return {};
}

// ---------------------------------------------------------------------------
// Cut form (CutSeg, CutWin).

struct HostCutSeg {
    int64_t a = 0, b = 0;  // rows
    bool has_lo = false, has_hi = false;  // a cut before / after it
    int same = -1;         // an earlier segment that is the same matrix, or -1
    SepHostPlan hp;
    SepPlan sp;
    std::vector<unsigned char> b64, b32;
};
struct HostCutWin {
    int64_t row = 0, first = 0;
    int same = -1;
    int len = 0;
    std::vector<double> w;  // [len][h]
};
struct HostCuts {
    std::vector<HostCutSeg> segs;
    std::vector<HostCutWin> wins;
};

// Rows c .. c + h - 1 of A^{-1} near their diagonal entries: the solutions of
// A^T w = e on the rows within kCutNear of the cut (the matrix beyond changes
// the entries kept below by the square of the decay over kCutNear rows).
// On either side entries w_i are dropped while two sums stay at most 2^-58 each:
// that of |w_i| in units of the row's largest, and that of |w_i| s_i, with s_i
// the largest coefficient of the matrix's row i, in units of the largest such
// term (1 if that is more).  The second does not change when a row and its
// right-hand sides are multiplied by the same factor, as the solution does not:
// with f = A x a right-hand side is at most (2h + 1) s_i max |x|, so what is
// dropped moves the unknown by at most (2h + 1) 2^-57 of the system's largest
// unknown.  (By |w_i| alone a row with a large diagonal entry, or large rows
// beside small ones, lost digits: diffusion n = 2500 with one entry 1e12 eleven
// rows before a cut, 4e-7.)  False if more than kMaxCutReach rows on a side are
// left.  Rows of a periodic matrix are counted round (n > 2 kCutNear + 1).
constexpr int64_t kCutNear = 256;

template <class M>
bool cut_window(bool periodic, int64_t n, const double *bands, int64_t row, HostCutWin &win) {
    constexpr int h = M::h;
    const int64_t lo = periodic ? row - kCutNear : std::max<int64_t>(0, row - kCutNear);
    const int64_t hi = periodic ? row + h + kCutNear : std::min<int64_t>(n, row + h + kCutNear), ns = hi - lo;
    std::vector<typename M::Row> rows(ns);
    int64_t bad = -1;
    auto wrapped = [&](int64_t r) { return r < 0 ? r + n : r >= n ? r - n : r; };
    // entry (i, i + k - h) of A^T is A's entry (i + k - h, i): band 2h - k of that row
    auto tr = [&](int k, int64_t i) -> double {
        const int64_t j = i + k - h;
        return j < 0 || j >= ns ? 0.0 : bands[(int64_t)(2 * h - k) * n + wrapped(lo + j)];
    };
    if (!M::factor(ns, tr, rows.data(), &bad)) return false;
    std::vector<double> v((size_t)h * ns, 0.0), scale(ns, 0.0);
    for (int64_t i = 0; i < ns; ++i)
        for (int k = 0; k < 2 * h + 1; ++k) {
            const int64_t r = lo + i, col = r + k - h;
            if (periodic || (col >= 0 && col < n))
                scale[i] = std::max(scale[i], std::fabs(bands[(int64_t)k * n + wrapped(r)]));
        }
    for (int c = 0; c < h; ++c) v[(row + c - lo) * h + c] = 1.0;
    M::template solve<h>(ns, rows.data(), v.data());
    int64_t reach_lo = 0, reach_hi = 0;
    for (int c = 0; c < h; ++c) {
        auto size = [&](int64_t i) { return std::fabs(v[i * h + c]); };
        double mx = 0.0, mxs = 0.0;
        for (int64_t i = 0; i < ns; ++i) {
            mx = std::max(mx, size(i));
            mxs = std::max(mxs, size(i) * scale[i]);
        }
        if (!std::isfinite(mx) || !std::isfinite(mxs)) return false;
        const double most = std::ldexp(mx, -58), mosts = std::ldexp(std::min(mxs, 1.0), -58);
        double s = 0.0, ss = 0.0;
        auto drops = [&](int64_t i) { return (s += size(i)) <= most && (ss += size(i) * scale[i]) <= mosts; };
        int64_t i = 0, e = ns - 1;
        while (i < row - lo && drops(i)) ++i;
        s = ss = 0.0;
        while (e > row + h - 1 - lo && drops(e)) --e;
        reach_lo = std::max(reach_lo, row - lo - i);
        reach_hi = std::max(reach_hi, lo + e - (row + h - 1));
    }
    if (reach_lo > kMaxCutReach || reach_hi > kMaxCutReach) return false;
    win.row = row;
    win.first = row - reach_lo;
    win.len = (int)(reach_lo + h + reach_hi);
    win.w.assign(v.begin() + (win.first - lo) * h, v.begin() + (win.first - lo + win.len) * h);
    return true;
}

// The cut form's own solve of the gate's columns, as the kernels run it.
template <class M>
void cut_solve(const HostCuts &hc, int64_t n, const double *bands, Columns &x) {
    constexpr int h = M::h, C = kChecks;
    for (size_t k = 0; k < hc.wins.size(); ++k) {
        const HostCutWin &w = hc.wins[k], &src = w.same >= 0 ? hc.wins[w.same] : w;
        double z[2][C] = {};
        for (int i = 0; i < src.len; ++i) {
            const double *f = x.data() + (w.first + i + n) % n * C;
            for (int c = 0; c < h; ++c)
                for (int q = 0; q < C; ++q) z[c][q] += src.w[(size_t)i * h + c] * f[q];
        }
        for (int c = 0; c < h; ++c) std::copy(z[c], z[c] + C, x.data() + (w.row + c) * C);
    }
    for (const HostCutSeg &s : hc.segs) {
        double *f = x.data() + s.a * C;
        const int64_t ns = s.b - s.a;
        for (int t = 0; t < h; ++t)
            for (int c = 0; c < h; ++c)
                for (int q = 0; q < C; ++q) {
                    if (s.has_lo && c >= t && t < ns)
                        f[t * C + q] -= bands[(int64_t)(c - t) * n + s.a + t] * x[(s.a - h + c + n) % n * C + q];
                    if (s.has_hi && c <= t)
                        f[(ns - h + t) * C + q] -=
                            bands[(int64_t)(2 * h + c - t) * n + s.b - h + t] * x[(s.b + c) * C + q];
                }
        sep_plan_solve<M>(s.same >= 0 ? hc.segs[s.same].hp : s.hp, false, ns, f);
    }
}

// Segments of `run` rows and cuts; the last segment takes what is left once that
// is no more than kCutRows.  For a periodic matrix the last cut is its last row.
std::vector<HostCutSeg> lay_cuts(int h, bool periodic, int64_t n, int64_t run) {
    std::vector<HostCutSeg> segs;
    const int64_t end = periodic ? n - h : n;
    for (int64_t a = 0; a < end;) {
        HostCutSeg s;
        s.a = a;
        s.b = end - a <= kCutRows ? end : a + run;
        s.has_lo = a > 0 || periodic;
        s.has_hi = s.b < n;
        a = s.b + h;
        // what is left after a cut has to be a segment: a last cut with none
        // after it leaves no rows to be solved by it
        if (s.b < end && a >= end) s.b = end, s.has_hi = s.b < n, a = end;
        segs.push_back(std::move(s));
    }
    return segs;
}

// Cuts the matrix into segments of at most kCutRows rows, all of them a whole
// number of 32-row blocks but the last: about equal ones, or shorter ones where
// the last would be longer or (periodic) too short for the windows of the cuts
// on either side.  False if a window is too wide, a plan is missing, or the
// result is not the recurrences' within kPlanTolerance.
template <class M>
bool build_cuts(bool periodic, int64_t n, const double *bands, const Gate &gate, HostCuts &hc) {
    constexpr int kind = M::kind, h = M::h;
    const int64_t Q = (n + h + kCutRows + h - 1) / (kCutRows + h);
    if (Q < 2 || Q > kMaxCutSegs || (periodic && n < 2 * kCutNear + 2)) return false;
    // the whole blocks nearest to an equal share from below, from above, then less
    const int64_t below = (n - h * (Q - 1)) / Q / kSegLb * kSegLb;
    std::vector<int64_t> runs = {below, below + kSegLb};
    for (int64_t run = below - kSegLb; run >= kCutRows / 2; run -= kSegLb) runs.push_back(run);
    for (int64_t run : runs) {
        if (run < kSegLb || run > kCutRows) continue;
        hc.segs = lay_cuts(h, periodic, n, run);
        hc.wins.clear();
        if ((int64_t)hc.segs.size() > kMaxCutSegs) return false;
        if (hc.segs.size() < 2 || hc.segs.back().b - hc.segs.back().a > kCutRows) continue;
        if (run == below && (int64_t)hc.segs.size() > Q) continue;  // one segment more than the fewest
        bool ok = true;
        for (const HostCutSeg &s : hc.segs) {
            if (!s.has_hi) continue;
            HostCutWin w;
            const int64_t row = s.b;
            // an earlier cut whose surroundings are the same has the same window
            for (size_t q = 0; q < hc.wins.size() && w.same < 0; ++q) {
                const HostCutWin &o = hc.wins[q];
                if (o.same >= 0 || o.row < kCutNear + h || row + 2 * h + kCutNear > n) continue;
                bool alike = true;
                for (int64_t i = -kCutNear - h; i < kCutNear + 2 * h && alike; ++i)
                    for (int b = 0; b < kind && alike; ++b) alike = bands[b * n + row + i] == bands[b * n + o.row + i];
                if (!alike) continue;
                w.same = (int)q;
                w.row = row;
                w.first = row + (o.first - o.row);
                w.len = o.len;
            }
            if (w.same < 0 && !cut_window<M>(periodic, n, bands, row, w)) return false;
            hc.wins.push_back(std::move(w));
        }
        // a window must not reach another cut: its rows are overwritten
        const size_t nw = hc.wins.size();
        for (size_t k = 0; k < nw && ok; ++k) {
            const HostCutWin &w = hc.wins[k];
            if (k > 0) ok = ok && w.first >= hc.wins[k - 1].row + h;
            if (k + 1 < nw) ok = ok && w.first + w.len <= hc.wins[k + 1].row;
            if (periodic && k == 0) ok = ok && w.first + n >= hc.wins[nw - 1].row + h;
            if (periodic && k + 1 == nw) ok = ok && w.first + w.len - n <= hc.wins[0].row;
        }
        if (ok) break;
        hc.segs.clear();
    }
    if (hc.segs.size() < 2) return false;
    std::vector<std::vector<double>> sub;
    for (HostCutSeg &s : hc.segs) {
        sub.push_back(sub_bands(kind, n, bands, s.a, s.b));
        for (size_t q = 0; q + 1 < sub.size() && s.same < 0; ++q)
            if (hc.segs[q].same < 0 && sub[q] == sub.back()) s.same = (int)q;
        if (s.same < 0 && !build_sep_plan<M>(false, s.b - s.a, sub.back().data(), kSegLb, nullptr, s.hp)) return false;
    }
    if (!passes(gate, [&](Columns &x) { cut_solve<M>(hc, n, bands, x); })) return false;
    for (HostCutSeg &s : hc.segs)
        if (s.same < 0) serialise_sep<typename M::Row, typename M::Row32>(s.hp, s.b64, s.b32, s.sp);
    return true;
}

// The device's view of a segment: plan blob (FP32) and the kernel's copy.
RefSeg make_seg(const SepPlan &sp, const unsigned char *b32, const unsigned char *rec, int64_t lo, int64_t rows,
                int64_t a, int64_t b) {
    RefSeg s{};
    s.fwd = reinterpret_cast<const float *>(rec + sp.refine.fwd);
    s.bwd = reinterpret_cast<const float *>(rec + sp.refine.bwd);
    s.spk = reinterpret_cast<const float *>(rec + sp.refine.spk);
    s.sinv = reinterpret_cast<const float *>(rec + sp.refine.sinv);
    s.scf = reinterpret_cast<const float *>(b32 + sp.fac_bytes32 + sp.spk_bytes32);
    s.band = reinterpret_cast<const double *>(rec + sp.refine.band);
    s.map = reinterpret_cast<const int *>(b32 + sp.fac_bytes32 + sp.spk_bytes32 + sp.scf_bytes32 + sp.sinv_bytes32);
    s.lo = (int32_t)lo;
    s.rows = (int32_t)rows;
    s.a = (int32_t)a;
    s.b = (int32_t)b;
    s.P = sp.P;
    s.Nr = sp.Nr;
    s.ldsinv = sp.refine.ldsinv;
    return s;
}

}  // namespace

// Builds every plan that exists for this matrix.  A plan that does not exist
// (too many blocks, a zero pivot inside a block, a singular interface
// system) only disables the partitioned variant for that block length.
sbs_status build_partitions(sbs_lhs *h, const double *bands) {
    std::vector<unsigned char> b64[3], b32[3], s64[3], s32[3], r32[3];
    size_t total = 0;
    // A periodic tridiagonal matrix is partitioned directly (the blocks are
    // plain tridiagonal; the wrap is one more interface pair).
    const bool periodic = h->kind == SBS_TRI_PERIODIC;
    const bool tri = h->kind == SBS_TRI || periodic;
    // (longer matrices have no plan of the whole and no cut form)
    const Gate gate = h->n <= (int64_t)kMaxCutSegs * (kCutRows + 2)
                          ? (tri ? make_gate<Tri>(periodic, h->n, bands) : make_gate<Penta>(false, h->n, bands))
                          : Gate();
    for (int q = 0; q < 3; ++q) {
        HostPlan hp;
        const int lb = kPartLbs[q];
        const bool ok = tri ? build_plan<Tri>(periodic, h->n, bands, lb, gate, hp)
                            : build_plan<Penta>(false, h->n, bands, lb, gate, hp);
        if (!ok) continue;
        PartPlan &pp = h->part[q];
        pp.periodic = periodic;
        if (tri)
            serialise<TriRow<double>, TriRow<float>>(hp, b64[q], b32[q], pp);
        else
            serialise<PentaRow<double>, PentaRow<float>>(hp, b64[q], b32[q], pp);
        pp.lb = hp.lb;
        pp.P = hp.P;
        pp.Nr = hp.Nr;
        pp.ok = true;
        total += align256(b64[q].size()) + align256(b32[q].size());
    }
    for (int q = 0; q < 3; ++q) {
        SepHostPlan hp;
        const int lb = kPartLbs[q];
        const bool ok = tri ? build_sep_plan<Tri>(periodic, h->n, bands, lb, &gate, hp)
                            : build_sep_plan<Penta>(false, h->n, bands, lb, &gate, hp);
        if (!ok) continue;
        SepPlan &sp = h->sep[q];
        sp.periodic = periodic;
        if (tri)
            serialise_sep<TriRow<double>, TriRow<float>>(hp, s64[q], s32[q], sp);
        else
            serialise_sep<PentaRow<double>, PentaRow<float>>(hp, s64[q], s32[q], sp);
        sp.ok = true;
        total += align256(s64[q].size()) + align256(s32[q].size());
        if (!periodic && lb >= 32) {
            if (tri)
                serialise_refine<TriRow<float>>(hp, s32[q], sp, SBS_TRI, h->n, bands, r32[q], sp.refine);
            else
                serialise_refine<PentaRow<float>>(hp, s32[q], sp, SBS_PENTA, h->n, bands, r32[q], sp.refine);
            total += r32[q].size();
        }
    }
    // Segments for the mixed-precision kernels: overlapping runs of rows, or the
    // 32-row separator plan itself where the whole matrix is one.
    std::vector<HostSeg> segs;
    if (!periodic && h->n > (int64_t)seg_half(h->kind) * kSegLb)
        segs = tri ? build_segments<Tri>(h->n, bands, gate) : build_segments<Penta>(h->n, bands, gate);
    for (const HostSeg &s : segs)
        if (s.same < 0) total += align256(s.b32.size()) + align256(s.rec.size());
    if (!segs.empty() && h->n <= kMaxWhole) {
        int64_t blocks = 0;
        for (const HostSeg &s : segs) blocks += (s.hi - s.lo + kSegLb - 1) / kSegLb;
        h->seg_small = !pays(h->kind, blocks, (h->n + kSegLb - 1) / kSegLb, false);
    }
    const bool whole = segs.empty() && !periodic && h->sep[1].ok && h->sep[1].P <= seg_max_blocks(h->kind);
    const size_t nseg = whole ? 1 : segs.size();
    total += align256(nseg * sizeof(RefSeg));
    HostCuts hc;
    if (h->n > kCutRows) {
        const bool ok = tri ? build_cuts<Tri>(periodic, h->n, bands, gate, hc)
                            : build_cuts<Penta>(false, h->n, bands, gate, hc);
        if (!ok) hc = HostCuts();
    }
    for (const HostCutSeg &s : hc.segs) total += align256(s.b64.size()) + align256(s.b32.size());
    for (const HostCutWin &w : hc.wins) total += align256(w.w.size() * 8);
    total += align256(hc.segs.size() * sizeof(CutSeg)) + align256(hc.wins.size() * sizeof(CutWin));
    if (total == 0) return SBS_OK;
    void *dev = nullptr;
    if (hipMalloc(&dev, total) != hipSuccess) return SBS_ERR_NO_MEMORY;
    h->pdev = dev;
    // everything is laid out in host memory and goes over in one copy (each
    // copy of its own costs about 10 us, as much as a small plan)
    std::vector<unsigned char> host(total, 0);
    unsigned char *base = static_cast<unsigned char *>(dev);
    size_t at = 0;
    auto put = [&](const void *src, size_t bytes) {
        unsigned char *d = base + at;
        copy_bytes(host.data() + at, src, bytes);
        at += align256(bytes);
        return d;
    };
    for (int q = 0; q < 3; ++q) {
        PartPlan &pp = h->part[q];
        if (!pp.ok) continue;
        pp.blob64 = put(b64[q].data(), b64[q].size());
        pp.blob32 = put(b32[q].data(), b32[q].size());
    }
    for (int q = 0; q < 3; ++q) {
        SepPlan &sp = h->sep[q];
        if (!sp.ok) continue;
        sp.blob64 = put(s64[q].data(), s64[q].size());
        sp.blob32 = put(s32[q].data(), s32[q].size());
        if (!r32[q].empty()) sp.refine.base = put(r32[q].data(), r32[q].size());
    }
    std::vector<RefSeg> table;
    if (whole) {
        const SepPlan &sp = h->sep[1];
        table.push_back(make_seg(sp, static_cast<const unsigned char *>(sp.blob32),
                                 static_cast<const unsigned char *>(sp.refine.base), 0, h->n, 0, h->n));
    }
    for (const HostSeg &s : segs) {
        if (s.same >= 0) {
            RefSeg t = table[s.same];
            t.lo = (int32_t)s.lo;
            t.a = (int32_t)s.a;
            t.b = (int32_t)s.b;
            table.push_back(t);
            continue;
        }
        const unsigned char *b32 = put(s.b32.data(), s.b32.size());
        const unsigned char *rec = put(s.rec.data(), s.rec.size());
        table.push_back(make_seg(s.sp, b32, rec, s.lo, s.hi - s.lo, s.a, s.b));
    }
    if (!table.empty()) {
        h->segs = reinterpret_cast<const RefSeg *>(put(table.data(), table.size() * sizeof(RefSeg)));
        h->nseg = (int)table.size();
        for (const RefSeg &s : table) {
            h->segP = std::max(h->segP, (int)s.P);
            h->segNr = std::max(h->segNr, (int)s.Nr);
        }
    }
    if (!hc.segs.empty()) {
        const int bw = tri ? 1 : 2;
        const int64_t n = h->n;
        std::vector<CutSeg> cs;
        std::vector<CutWin> cw;
        for (const HostCutSeg &s : hc.segs) {
            CutSeg t{};
            if (s.same >= 0) {
                t = cs[s.same];
            } else {
                t.blob[0] = put(s.b64.data(), s.b64.size());
                t.blob[1] = put(s.b32.data(), s.b32.size());
                t.fac[0] = (int32_t)s.sp.fac_bytes64, t.fac[1] = (int32_t)s.sp.fac_bytes32;
                t.spk[0] = (int32_t)s.sp.spk_bytes64, t.spk[1] = (int32_t)s.sp.spk_bytes32;
                t.scf[0] = (int32_t)s.sp.scf_bytes64, t.scf[1] = (int32_t)s.sp.scf_bytes32;
                t.sinv[0] = (int32_t)s.sp.sinv_bytes64, t.sinv[1] = (int32_t)s.sp.sinv_bytes32;
                t.map = (int32_t)s.sp.map_bytes;
                t.P = s.sp.P;
                t.Nr = s.sp.Nr;
                t.kofs = s.sp.kofs;
                t.kw = s.sp.kw;
                h->cut.P = std::max(h->cut.P, s.sp.P);
                h->cut.Nr = std::max(h->cut.Nr, s.sp.Nr);
                for (int tc = 0; tc < 2; ++tc)
                    h->cut.blob_bytes[tc] = std::max(h->cut.blob_bytes[tc], s.sp.blob_bytes(tc));
            }
            t.row0 = (int32_t)s.a;
            t.rows = (int32_t)(s.b - s.a);
            t.has_lo = s.has_lo;
            t.has_hi = s.has_hi;
            t.lo_at = s.a > 0 ? -bw : (int32_t)(n - bw);
            t.hi_cut = (int32_t)cs.size();
            t.lo_cut = s.a > 0 ? t.hi_cut - 1 : (int32_t)hc.wins.size() - 1;
            for (int r = 0; r < 2; ++r)
                for (int c = 0; c < 2; ++c) {
                    t.lo[r][c] = t.hi[r][c] = 0.0;
                    if (r >= bw || c >= bw) continue;
                    if (t.has_lo && c >= r && r < t.rows) t.lo[r][c] = bands[(int64_t)(c - r) * n + s.a + r];
                    if (t.has_hi && c <= r) t.hi[r][c] = bands[(int64_t)(2 * bw + c - r) * n + s.b - bw + r];
                }
            cs.push_back(t);
        }
        for (const HostCutWin &w : hc.wins) {
            CutWin t{};
            t.w = w.same >= 0 ? cw[w.same].w : reinterpret_cast<const double *>(put(w.w.data(), w.w.size() * 8));
            t.row = (int32_t)w.row;
            t.first = (int32_t)((w.first + n) % n);
            t.len = w.len;
            cw.push_back(t);
        }
        h->cut.segs = reinterpret_cast<const CutSeg *>(put(cs.data(), cs.size() * sizeof(CutSeg)));
        h->cut.wins = reinterpret_cast<const CutWin *>(put(cw.data(), cw.size() * sizeof(CutWin)));
        h->cut.rows = cs.front().rows;
        h->cut.last = cs.back().rows;
        h->cut.Q = (int)cs.size();
        h->cut.cuts = (int)cw.size();
    }
    if (hipMemcpy(dev, host.data(), total, hipMemcpyHostToDevice) != hipSuccess) return SBS_ERR_DEVICE;
    h->device_bytes += (int64_t)total;
    return SBS_OK;
}

}  // namespace sbs
