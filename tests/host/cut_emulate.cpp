// Runs the cut form of a plain solve and the segments of the mixed-precision
// solve on the host, from the tables that build_partitions uploads (CutWin,
// CutSeg, RefSeg; the CPU stand-in for the device keeps them in host memory),
// step for step as the kernels do, with the indices they form checked.
//   cut_emulate in.bin out.bin
// in:  int32 kind, int64 n, int64 m, bands (3 or 5 x n doubles), rhs (n x m)
// out: int32 segments and cuts of the cut form (0: it has none), then (if it
//      has) the n x m FP64 solution; int32 segments of the mixed-precision
//      form, then (if there are any) its n x m solution (two corrections)
#define main part_emulate_main
#include "part_emulate.cpp"
#undef main

namespace {

void need(bool ok, const char *what) {
    if (ok) return;
    std::fprintf(stderr, "cut_emulate: %s\n", what);
    std::exit(4);
}

template <typename Row, typename Solve>
void emulate_cut(const sbs_lhs &h, const double *rhs, int64_t m, double *x, Solve solve) {
    const int H = h.kind == SBS_PENTA ? 2 : 1;
    const int64_t n = h.n;
    std::copy(rhs, rhs + n * m, x);
    std::vector<int> cut_of((size_t)n, -1);
    for (int k = 0; k < h.cut.cuts; ++k)
        for (int c = 0; c < H; ++c) {
            const int64_t r = h.cut.wins[k].row + c;
            need(r >= 0 && r < n && cut_of[r] < 0, "a cut's rows");
            cut_of[r] = k;
        }
    // the unknowns of the cut rows, in place of their right-hand sides
    for (int k = 0; k < h.cut.cuts; ++k) {
        const CutWin &w = h.cut.wins[k];
        need(w.first >= 0 && w.first < n && w.len >= H && w.len <= n, "a window's rows");
        for (int64_t j = 0; j < m; ++j) {
            double z[2] = {0.0, 0.0};
            for (int i = 0; i < w.len; ++i) {
                const int64_t r = w.first + i < n ? w.first + i : w.first + i - n;
                need(h.kind == SBS_TRI_PERIODIC || w.first + i < n, "a window past the last row");
                need(cut_of[r] < 0 || cut_of[r] == k, "a window holds another cut's row");
                for (int c = 0; c < H; ++c) z[c] = std::fma(w.w[i * H + c], rhs[r * m + j], z[c]);
            }
            for (int c = 0; c < H; ++c) x[(w.row + c) * m + j] = z[c];
        }
    }
    // the segments
    std::vector<char> done((size_t)n, 0);
    for (int k = 0; k < h.cut.Q; ++k) {
        const CutSeg &s = h.cut.segs[k];
        need(s.row0 >= 0 && s.rows >= 1 && s.row0 + s.rows <= n, "a segment's rows");
        need(s.rows == (k + 1 < h.cut.Q ? h.cut.rows : h.cut.last), "a segment's length");
        need(s.P <= h.cut.P && s.Nr <= h.cut.Nr, "a segment's plan");
        std::vector<double> f((size_t)s.rows * m), g(f.size());
        std::copy(x + (int64_t)s.row0 * m, x + (int64_t)(s.row0 + s.rows) * m, f.begin());
        const int64_t lo = s.row0 + s.lo_at, hi = s.row0 + s.rows;
        if (s.has_lo) need(lo >= 0 && cut_of[lo] == s.lo_cut && h.cut.wins[s.lo_cut].row == lo, "the cut before");
        if (s.has_hi) need(hi < n && cut_of[hi] == s.hi_cut && h.cut.wins[s.hi_cut].row == hi, "the cut after");
        // (the kernel keeps both cuts' unknowns for one-row cuts only, and a ragged
        // last block meets a cut only there)
        need(H == 1 || !s.has_hi || (s.rows % kSegLb == 0 && (!s.has_lo || s.P > 1)), "both cuts of a lane");
        for (int64_t j = 0; j < m; ++j)
            for (int t = 0; t < H; ++t)
                for (int c = 0; c < H; ++c) {
                    if (s.has_lo && c >= t && t < s.rows) f[t * m + j] -= s.lo[t][c] * x[(lo + c) * m + j];
                    if (s.has_hi && c <= t) f[(s.rows - H + t) * m + j] -= s.hi[t][c] * x[(hi + c) * m + j];
                }
        SepPlan sp;
        sp.lb = kSegLb;
        sp.P = s.P;
        sp.Nr = s.Nr;
        sp.kofs = s.kofs;
        sp.kw = s.kw;
        sp.blob64 = const_cast<unsigned char *>(s.blob[0]);
        sp.fac_bytes64 = s.fac[0];
        sp.spk_bytes64 = s.spk[0];
        sp.scf_bytes64 = s.scf[0];
        sp.sinv_bytes64 = s.sinv[0];
        sbs_lhs part;
        part.kind = H == 2 ? SBS_PENTA : SBS_TRI;
        part.n = s.rows;
        emulate_sep<Row>(part, sp, f.data(), m, g.data(), solve);
        std::copy(g.begin(), g.end(), x + (int64_t)s.row0 * m);
        std::fill(done.begin() + s.row0, done.begin() + s.row0 + s.rows, 1);
    }
    for (int64_t i = 0; i < n; ++i) need(done[i] != (cut_of[i] >= 0), "a row solved by nothing, or twice");
}

void emulate_segs(const sbs_lhs &h, const double *rhs, int64_t m, double *x) {
    int64_t next = 0;
    for (int k = 0; k < h.nseg; ++k) {
        const RefSeg &s = h.segs[k];
        need(s.a == next && s.lo <= s.a && s.b <= s.lo + s.rows && s.lo >= 0 && s.lo + s.rows <= h.n, "a segment's rows");
        need(s.P <= h.segP && s.Nr <= h.segNr, "a segment's plan");
        next = s.b;
        SepPlan sp;
        sp.lb = kSegLb;
        sp.P = s.P;
        sp.Nr = s.Nr;
        const unsigned char *rec = reinterpret_cast<const unsigned char *>(s.fwd);
        auto at = [&](const void *p) { return (size_t)(static_cast<const unsigned char *>(p) - rec); };
        sp.refine.base = const_cast<unsigned char *>(rec);
        sp.refine.fwd = 0;
        sp.refine.bwd = at(s.bwd);
        sp.refine.spk = at(s.spk);
        sp.refine.band = at(s.band);
        sp.refine.sinv = at(s.sinv);
        sp.refine.ldsinv = s.ldsinv;
        const unsigned char *scf = reinterpret_cast<const unsigned char *>(s.scf);
        sp.blob32 = const_cast<unsigned char *>(scf);
        sp.scf_bytes32 = (size_t)(reinterpret_cast<const unsigned char *>(s.map) - scf);
        sbs_lhs part;
        part.kind = h.kind;
        part.n = s.rows;
        std::vector<double> g((size_t)s.rows * m);
        emulate_refine(part, sp, rhs + (int64_t)s.lo * m, m, g.data());
        std::copy(g.begin() + (int64_t)(s.a - s.lo) * m, g.begin() + (int64_t)(s.b - s.lo) * m, x + (int64_t)s.a * m);
    }
    need(next == h.n, "the last segment's end");
}

}  // namespace

int main(int argc, char **argv) {
    if (argc != 3) return 2;
    FILE *f = std::fopen(argv[1], "rb");
    if (!f) return 2;
    int32_t kind;
    int64_t n, m;
    if (std::fread(&kind, 4, 1, f) != 1 || std::fread(&n, 8, 1, f) != 1 || std::fread(&m, 8, 1, f) != 1) return 2;
    const int nb = kind == SBS_TRI_PERIODIC ? 3 : kind;
    std::vector<double> bands((size_t)nb * n), rhs((size_t)n * m), x((size_t)n * m);
    if (std::fread(bands.data(), 8, bands.size(), f) != bands.size()) return 2;
    if (std::fread(rhs.data(), 8, rhs.size(), f) != rhs.size()) return 2;
    std::fclose(f);
    sbs_lhs h;
    h.kind = kind;
    h.n = n;
    if (build_partitions(&h, bands.data()) != SBS_OK) return 3;
    FILE *o = std::fopen(argv[2], "wb");
    if (!o) return 2;
    const int32_t cut[2] = {h.cut.Q, h.cut.cuts};
    std::fwrite(cut, 4, 2, o);
    if (h.cut.Q) {
        if (kind != SBS_PENTA)
            emulate_cut<TriRow<double>>(h, rhs.data(), m, x.data(), solve_tri_rows);
        else
            emulate_cut<PentaRow<double>>(h, rhs.data(), m, x.data(), solve_penta_rows);
        std::fwrite(x.data(), 8, x.size(), o);
    }
    const int32_t nseg = h.nseg;
    std::fwrite(&nseg, 4, 1, o);
    if (nseg) {
        emulate_segs(h, rhs.data(), m, x.data());
        std::fwrite(x.data(), 8, x.size(), o);
    }
    std::fclose(o);
    if (h.pdev) std::free(h.pdev);
    return 0;
}
