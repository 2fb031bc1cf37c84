// C-ABI entry points: argument checking, the host-side FP64 factorisation of
// the shared matrix, its upload, and dispatch to the HIP kernels.
#include <atomic>
#include <climits>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <tuple>
#include <vector>

#include "factor_rows.h"
#include "internal.h"

using namespace sbs;

namespace {

// Coefficient k of row i of a row-aligned band array, 0 outside the matrix.
double coef(const double *bands, int kind, int64_t n, int k, int64_t i) {
    const int64_t col = i + k - kind / 2;
    if (col < 0 || col >= n) return 0.0;
    return bands[(int64_t)k * n + i];
}

template <typename Row32, typename Row64>
Row32 narrow(const Row64 &r);
template <>
TriRow<float> narrow(const TriRow<double> &r) {
    return {(float)r.a_s, (float)r.chat, (float)r.inv, 0.0f};
}
template <>
PentaRow<float> narrow(const PentaRow<double> &r) {
    return {(float)r.eps_s, (float)r.beta_s, (float)r.inv, (float)r.gamma, (float)r.delta, 0.f, 0.f, 0.f};
}
template <>
PeriodicRow<float> narrow(const PeriodicRow<double> &r) {
    return {(float)r.a_s, (float)r.chat, (float)r.inv, (float)r.wt, (float)r.z, 0.f, 0.f, 0.f};
}

int nbands(int kind) { return kind == SBS_TRI_PERIODIC ? 3 : kind; }

// Whether each band holds one value wherever it lies inside the matrix (every
// row of a periodic matrix); if so, those values.  A band with no entry inside
// (a penta band of a 1-row matrix) counts as constant 0.
bool constant_bands(const double *bands, int kind, int64_t n, BandCoef *c) {
    const int nb = nbands(kind), H = nb / 2;
    for (int k = 0; k < nb; ++k) {
        bool have = false;
        c->c[k] = 0.0;
        for (int64_t i = 0; i < n; ++i) {
            const int64_t col = i + k - H;
            if (kind != SBS_TRI_PERIODIC && (col < 0 || col >= n)) continue;
            const double v = bands[(int64_t)k * n + i];
            if (!have) {
                c->c[k] = v;
                have = true;
            } else if (v != c->c[k]) {
                return false;
            }
        }
    }
    return true;
}

// Band k of row i as the matrix uses it: 0 outside a banded matrix; every
// entry (the corners a_0 and c_{n-1} included) for a periodic one.
double entry(const double *bands, int kind, int64_t n, int k, int64_t i) {
    return kind == SBS_TRI_PERIODIC ? bands[(int64_t)k * n + i] : coef(bands, kind, n, k, i);
}

template <typename Row64, typename Row32>
sbs_status upload(sbs_lhs *h, const std::vector<Row64> &r64, const double *B) {
    const int64_t rows = h->rows;
    const size_t b64 = sizeof(Row64) * rows, b32 = sizeof(Row32) * rows, bb = sizeof(BandRow) * rows;
    const size_t total = b64 + b32 + bb;
    std::vector<unsigned char> host(total, 0);  // padding rows stay zero
    std::memcpy(host.data(), r64.data(), sizeof(Row64) * h->n);
    Row32 *p32 = reinterpret_cast<Row32 *>(host.data() + b64);
    for (int64_t i = 0; i < h->n; ++i) p32[i] = narrow<Row32>(r64[i]);
    BandRow *pb = reinterpret_cast<BandRow *>(host.data() + b64 + b32);
    for (int64_t i = 0; i < h->n; ++i)
        for (int k = 0; k < nbands(h->kind); ++k) pb[i].c[k] = entry(B, h->kind, h->n, k, i);

    if (hipGetDevice(&h->device) != hipSuccess) return SBS_ERR_DEVICE;
    void *dev = nullptr;
    if (hipMalloc(&dev, total) != hipSuccess) return SBS_ERR_NO_MEMORY;
    if (hipMemcpy(dev, host.data(), total, hipMemcpyHostToDevice) != hipSuccess) {
        (void)hipFree(dev);
        return SBS_ERR_DEVICE;
    }
    h->dev = dev;
    h->fac64 = dev;
    h->fac32 = static_cast<unsigned char *>(dev) + b64;
    h->bands = reinterpret_cast<BandRow *>(static_cast<unsigned char *>(dev) + b64 + b32);
    h->device_bytes = (int64_t)total;
    return SBS_OK;
}

bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

// Which partitioned form runs: the separator kernel when it fills the GPU
// with whole row runs from a plan in LDS; else the pair kernel; else a
// separator shape (for AUTO only one whose plan sits in LDS or whose row
// runs are at least 128 bytes: a plan read from global memory with shorter
// runs loses to the chunked sweep).  A plan read from global memory loses
// to the pair form (random-band pentadiagonal n = 1024: 263.6 us against
// 225.6 us), so it runs only where the pair form has no plan.
// 0: none (AUTO then runs the sweeps), 1: separator, 2: pair.
int pick_uncached(const sbs_lhs *h, int t, int64_t m, const void *rhs, bool for_auto, sbs::SepChoice *sc,
                  sbs::PartChoice *pc) {
    const bool sep = sbs::choose_sep(h, t, m, rhs, sc);
    const bool part = sbs::choose_partition(h, t, m, pc);
    if (sep && !sc->gf && sbs::sep_fills(h, t, m, *sc)) return 1;
    // too few systems to fill the chip with whole row runs: where the pair
    // form would take 64-row blocks of at most 16 systems (128-byte runs),
    // the separator form's 32-row blocks with two systems per lane and 16
    // per workgroup (plan in LDS) finish sooner (tridiagonal n = 2048,
    // m = 2048: 15.4 against 19.0 us; pentadiagonal n = 1024, m = 2048: 11.7
    // against 16.5 us; tridiagonal n = 2048, m = 8192: 63.7 against
    // 67.8 us); against shorter pair blocks it was not faster throughout,
    // and where the pair form has 256-byte runs those are worth more
    if (part && t == 0 && h->part[pc->plan].lb == 64 && pc->S <= 16) {
        sbs::SepChoice alt;
        if (sbs::sep_shape(h, t, m, rhs, 32, 2, 16, 0, &alt) && !alt.gf) {
            *sc = alt;
            return 1;
        }
    }
    // pentadiagonal, where the pair form would take 32-row blocks of at most
    // 16 systems: 16-row separator blocks, one system per lane, 16 per
    // workgroup (n = 512, m = 4096: 10.0 against 11.7 us; n = 384,
    // m = 2048: 8.7 against 10.2 us; n = 512, m = 1024: 8.9 against 9.5 us;
    // for tridiagonal matrices the two were even)
    if (part && t == 0 && h->kind == SBS_PENTA && h->part[pc->plan].lb == 32 && pc->S <= 16) {
        sbs::SepChoice alt;
        if (sbs::sep_shape(h, t, m, rhs, 16, 1, 16, 0, &alt) && !alt.gf) {
            *sc = alt;
            return 1;
        }
    }
    if (part) return 2;
    const size_t elem = t == 0 ? 8 : 4;
    if (sep && (!for_auto || !sc->gf || (size_t)sc->S * elem >= 128)) return 1;
    return 0;
}

// Whether AUTO takes the cut form (two kernels, segments of 256 rows in runs of
// up to 1 KiB) instead of `form`.  Times are whole form against cut form.
//  - Always where a workgroup cannot hold a whole system with its plan in LDS:
//    the sweeps run one lane per system (pentadiagonal n = 5000, m = 500: 427
//    against 25 us; tridiagonal n = 8192, m = 4096: 618 against 116 us) and a
//    plan in memory costs a trip per block (pentadiagonal n = 1500 with random
//    bands, m = 2048: 127 against 24 us).
//  - Past 2048 rows always: pair and separator forms have runs of a few systems
//    and 30 to 500 us of latency (m = 500, tridiagonal n = 3000 64 against 21
//    us, pentadiagonal 73 and 23; n = 4096, m = 2048 40 and 33, 96 and 36 us).
//    From 1025 rows on where the separator form's runs are under 128 bytes and
//    there are systems enough for the cut form's (pentadiagonal n = 1600,
//    m = 1500: 40 against 26 us, n = 1300 with varying bands 42 and 24 us; FP32,
//    constant bands, n = 1536: m = 128 13 and 16 us, m = 500 37 and 19), or
//    its last round of workgroups is nearly empty and the cut form is one round
//    (m = 4400: pentadiagonal n = 1800, 245 workgroups, 34 against 31 us,
//    tridiagonal, 280, 31 and 38 us), and for the pair form, pentadiagonal FP64
//    (n = 1200 with varying bands, m = 1500: 50 against 25 us, m = 64 22 and
//    16 us) or while they stay in the cache below from 1729 on, in FP32 from eight
//    segments on and unless the pair form's workgroups are nearly a whole round, or
//    part of one with rows at whole cache lines (tridiagonal FP32 n = 1950, m = 777:
//    21 against 14 us, m = 6000 26 and 26, m = 8000 29 and 32; n = 1920, m = 4096 18
//    and 20, m = 5000 31 and 25; n = 1600, m = 777 17 and 19, n = 1792 periodic,
//    m = 1000 18 and 21).
//  - Else never for what stays in the 256 MB memory-side cache from one launch to
//    the next (n = 1000, m = 8192: 24 against 31 us; n = 2000, m = 4096: 30
//    against 31 us; from 98 MB on, n = 1500, m = 8192: 50 against 46 us).
//  - From 1025 rows on by where the whole form's 128-byte runs lie.  In rows that
//    start at multiples of 128 bytes a run is one cache line (m = 20000:
//    tridiagonal n = 1500 104 against 110 us, n = 2048 138 and 143 us,
//    pentadiagonal n = 1300 97 and 111, n = 1900 138 and 146 us), in others part
//    of two (m = 25000: 153 and 141, 205 and 186, 140 and 136, 198 and 184 us);
//    rows a multiple of 128 KiB apart (64 KiB from 1857 rows on) put a system's
//    blocks into few memory channels (m = 16384: 109 and 91, 148 and 113, 99 and
//    90, 147 and 118 us).  So for lines, other rows apart, the whole form; but not
//    with fewer lanes than 47 blocks of FP64 (37 of FP32) make, tridiagonal
//    (n = 1100, m = 20000: 97 and 87 us, n = 1300 112 and 103 us; FP32 n = 1100,
//    m = 40000 87 and 84 us, n = 1300 98 and 103 us), and not for pentadiagonal
//    band rows (n = 1100, m = 20000: 102 and 94 us) or, in FP32, up to 1984 rows
//    (band rows 1856; m = 40000: n = 1700 164 and 134 us, n = 1900 187 and 160,
//    n = 2048 157 and 161; band rows n = 1700 165 and 136, n = 1900 154 and 159).
//    Up to 1024 rows in FP32 from 601 rows on (tridiagonal n = 768, m = 160000:
//    322 against 226 us; n = 512: 176 against 187 us).
//  - Odd batches the whole form reads 8 (4) bytes per lane (n = 700, m = 99999:
//    338 against 281, 362 against 288 us); from 449 rows on in FP64 tridiagonal
//    (260 MB: n = 480 129 against 118 us, n = 400 122 against 127), else from
//    321 (pentadiagonal FP32 n = 343 151 against 142 us, n = 270 159 and 177).
//  - FP64 up to 1024 rows the whole form reads everything once in 256-byte runs
//    (n = 768, m = 60000: 149 against 154 us).  With rows a multiple of 128 KiB
//    apart its 32 blocks of 32 rows meet in few memory channels, where the cut
//    form's four segments are full ones (from 1009 rows on, tridiagonal from 993
//    on; states in rotation, n = 1024, m = 32768, 49152 and 65536: tridiagonal 121
//    against 111 us, 177 and 168, 243 and 221, pentadiagonal 118 and 116, 175 and
//    174, 240 and 227, with band rows 126 and 117, 180 and 175, 258 and 227; past
//    512 MiB even: m = 81920 297 and 293, 297 and 300; n = 1000: tridiagonal 116
//    and 115, 172 and 170, 236 and 220, pentadiagonal m = 32768 114 and 120;
//    n = 961, m = 49152: 165 and 167, 164 and 179; other rows apart: n = 1024,
//    m = 60000 212 and 221).
//
// cc: the cut form's shape for these systems.
bool takes_cut(const sbs_lhs *h, int t, int64_t m, const void *rhs, int form, const sbs::SepChoice &sc,
               const sbs::PartChoice &pc, const sbs::CutChoice &cc) {
    if (form == 0 || (form == 1 && sc.gf) || h->n > 2048) return true;
    const int64_t elem = t == 0 ? 8 : 4, pitch = m * elem, bytes = h->n * pitch;
    const int64_t cus = device_cus(h->device);
    if (h->n > 1024) {
        if (form == 2 && t == 0 && (h->kind == SBS_PENTA || (h->n > 1728 && bytes < 90000000))) return true;
        if (form == 2 && t == 1 && h->n > 1798 && bytes < 90000000) {
            const bool one_round = (m + pc.S - 1) / pc.S <= cus;
            if (!(one_round && (m > 24 * cus || (m >= 8 * cus && pitch % 128 == 0)))) return true;
        }
        if (form == 1 && sc.S * elem < 128 && m >= (t == 1 && h->constant_bands ? 256 : 128)) return true;
        const int64_t at_once = cus * std::max(1, sc.wgs), groups = form == 1 ? (m + sc.S - 1) / sc.S : 0;
        const int64_t cut_wgs = (m + cc.S - 1) / cc.S * h->cut.Q;
        if (form == 1 && groups > at_once && groups * 4 <= at_once * 5 && (t == 1 || cut_wgs <= cus * cc.wgs)) return true;
    }
    if (bytes < 90000000) return false;
    if (h->n > 1024) {
        const bool lines = (form == 1 ? sc.S : pc.S) * elem >= 128 && pitch % 128 == 0;
        if (!lines || pitch % (128 * 1024) == 0 || (pitch % (64 * 1024) == 0 && h->n > 1856)) return true;
        if (h->kind == SBS_PENTA) return t == 0 ? !h->constant_bands : h->n <= (h->constant_bands ? 1984 : 1856);
        return h->n <= (t == 0 ? 46 * 32 : 36 * 32);
    }
    if (bytes < int64_t(1) << 27) return false;
    if (m % 2 || !aligned(rhs, 2 * elem)) return h->n > (t == 0 && h->kind != SBS_PENTA ? 448 : 320);
    if (t == 1) return h->n > 600;
    return h->n > (h->kind == SBS_PENTA ? 1008 : 992) && pitch % (128 * 1024) == 0 && bytes <= int64_t(1) << 29;
}

// The choice depends on the handle, the dtype, m, whether rhs is aligned for
// two systems per lane and AUTO or not; it is made once and kept (weighing
// every shape costs several microseconds, as much as a small solve).
//
// cut (optional): the cut form where AUTO takes it instead (takes_cut); S 0 if
// it does not.  The queries report the whole-system form.
int pick_partition(const sbs_lhs *h, int t, int64_t m, const void *rhs, bool for_auto, sbs::SepChoice *sc,
                   sbs::PartChoice *pc, sbs::CutChoice *cut = nullptr) {
    struct Pick {
        int form;
        sbs::SepChoice sc;
        sbs::PartChoice pc;
        sbs::CutChoice cut;
    };
    static std::mutex mu;
    static std::map<std::tuple<uint64_t, int, int64_t, bool, bool>, Pick> known;
    const bool al = reinterpret_cast<uintptr_t>(rhs) % (2 * (t == 0 ? 8 : 4)) == 0;
    const auto key = std::make_tuple(h->id, t, m, al, for_auto);
    {
        std::lock_guard<std::mutex> g(mu);
        auto it = known.find(key);
        if (it != known.end()) {
            *sc = it->second.sc;
            *pc = it->second.pc;
            if (cut) *cut = it->second.cut;
            return it->second.form;
        }
    }
    const int form = pick_uncached(h, t, m, rhs, for_auto, sc, pc);
    sbs::CutChoice cc;
    if (for_auto && sbs::choose_cut(h, t, m, &cc) && !takes_cut(h, t, m, rhs, form, *sc, *pc, cc)) cc = sbs::CutChoice();
    if (cut) *cut = cc;
    std::lock_guard<std::mutex> g(mu);
    if (known.size() >= 4096) known.clear();  // bounded: many batch sizes only cost a new choice
    try {
        known[key] = Pick{form, *sc, *pc, cc};
    } catch (const std::bad_alloc &) {  // chosen again next time
    }
    return form;
}

// Whether a Crank-Nicolson call of one step takes the cut form although other
// forms fit.
// It crosses HBM once per step, the others once per call, so only for one step
// (several are then the same arithmetic however a caller groups them): past
// 2048 rows, where the pair form (constant bands) has short row runs and few
// waves (diffusion n = 2500, m = 8192: 92 against 122 us, four steps 321 and
// 187 us; n = 4000, m = 2000: 38 and 44 us, 145 and 64 us), and with band rows
// where those fill LDS (tridiagonal n = 2000, m = 2000: 31 against 66 us;
// n = 600, m = 100000: 254 and 327 us; n = 1000, m = 8192: 41 and 42 us,
// m = 1000: 30 and 20 us; constant bands n = 1000, m = 60000: 236 and 222 us).
// Pentadiagonal matrices have no pair form past 1792 rows, and 8 systems per
// workgroup in the separator form (constant bands, n = 2000: m = 500 28 against
// 26 us, m = 4096 47 and 42, m = 32768 452 and 277, the sweeps 345).
//
// pc: the pair form's shape, if it has one (null: not).  For tridiagonal
// matrices that keeps its single launch where the cut form's second one, or its
// rounds of workgroups, cost more (whole form against cut form):
//  - constant bands on up to three quarters of the CUs (n = 2500: m = 64 19
//    against 24 us, m = 500 27 and 29, m = 1000 36 and 31; n = 2221, m = 682 30
//    and 32), and up to 2176 rows for the 3000 to
//    8192 systems that make few rounds of the cut form's 9 segments (periodic
//    n = 2112: m = 4000 53 and 62, m = 8000 105 and 114; n = 2100: 55 and 57, 107
//    and 104, m = 2000 48 and 35, m = 16000 223 and 194);
//  - band rows of at most 1728 rows in FP64 with 16 systems per workgroup while
//    these are one round, from 1537 rows on two (n = 1030: m = 500 20 against
//    29 us, m = 4000 28 and 33, m = 16000 96 and 84; n = 1728: m = 4000 37 and
//    39, m = 8000 65 and 75; n = 1150, m = 8000 65 and 55; n = 1514, m = 6000 64 and
//    55).  A last block that is not full runs row by row; without one, from 1280
//    rows on, up to three rounds where the cut form makes as many (n = 1472:
//    m = 5000, one round for two, 51 and 39 us, m = 6000, two, 50 and 55,
//    m = 10000, two for three, 76 and 65, m = 12000, three, 82 and 85, m = 16000
//    110 and 100; n = 1216, m = 8000 56 and 54).  With fewer systems up to 1536
//    rows and half the CUs (n = 1300: m = 500 27 and 29, m = 1000 35 and 29;
//    n = 1800: m = 64 27 and 23);
//  - band rows in FP32 up to 1000 systems (n = 1450: m = 500 22 and 28; n = 1600:
//    m = 4000 37 and 31; n = 1553, m = 1100 32 and 27; n = 2000: m = 500 35 and
//    27), with whole 64-row blocks up to 5 systems a CU (n = 1600, m = 1100 29 and
//    31), and from 1150 rows on with 32-row blocks while the workgroups are one
//    round (n = 1408: m = 1500 24 and 30, m = 3000 25 and 32, m = 4400 34 and 33;
//    n = 1100, m = 2000 34 and 26), past 6 systems a CU only with a last block
//    that is whole or up to half full (n = 1411, m = 4096 25 and 28, n = 1406 32
//    and 28, n = 1207, m = 1100 25 and 30);
//  - large batches of fewer than 384 rows in FP64 (n = 300, m = 100000: 148
//    against 157 us; n = 400: 186 and 175), and of 769 to 960 rows under 300 MB,
//    whose workgroups of 32 systems are 800 lanes or more (n = 800: m = 32768
//    115 against 126 us, m = 50000 183 and 181; n = 900: m = 32768 126 and 131,
//    m = 50000 206 and 188; n = 700: m = 32768 131 and 104, n = 1000: 179 and 138).
bool takes_cut_cn(const sbs_lhs *h, int t, int64_t m, const sbs::PartChoice *pc, const sbs::CutChoice &cc) {
    const int64_t bytes = h->n * m * (t == 0 ? 8 : 4);
    if (!(h->n > 2048 || (h->kind == SBS_PENTA && h->n > 1792) ||
          (!h->constant_bands && (h->n > 1024 || bytes >= int64_t(1) << 27))))
        return false;
    if (!pc || h->kind == SBS_PENTA) return true;
    if (h->n <= 1024) return t == 1 || (h->n >= 384 && !(h->n > 768 && h->n <= 960 && bytes < 300000000));
    const int64_t cus = device_cus(h->device), groups = (m + pc->S - 1) / pc->S;
    if (h->constant_bands) return groups > cus * 3 / 4 && !(h->n <= 2176 && m >= 3000 && m <= 8192);
    const int lb = h->part[pc->plan].lb;
    const int64_t ragged = h->n % lb;
    if (t == 1) {
        if (h->n > 1728) return true;
        if (h->n >= 1150 && lb == 32 && (ragged <= 16 || m <= 6 * cus)) return groups > cus;
        return m > (lb == 64 && !ragged ? std::max<int64_t>(1000, 5 * cus) : 1000);
    }
    if (pc->S >= 16 && ragged) return h->n > 1728 || groups > cus * (h->n > 1536 ? 2 : 1);
    if (pc->S >= 16) {
        const int64_t slots = cus * cc.wgs, cut_rounds = ((m + cc.S - 1) / cc.S * h->cut.Q + slots - 1) / slots;
        const int64_t rounds = (groups + cus - 1) / cus;
        return h->n > 1728 || (rounds > 1 && (h->n < 1280 || rounds > 3 || cut_rounds < rounds));
    }
    return h->n > 1536 || groups > cus / 2;
}

// How a Crank-Nicolson call runs: the form, and the kernels' variant (cn: 1 band
// rows, 2 constant bands by value with no band rows in LDS, 3 see launch_partition).
struct CnChoice {
    enum Form { sweeps, separator, pair, cut } form = sweeps;
    int cn = 1;
    SepChoice sc;
    PartChoice pc;
    CutChoice cc;
};

CnChoice choose_cn(const sbs_lhs *h, int t, int64_t m, const void *c, int steps, bool cut_ok) {
    CnChoice k;
    k.cn = h->constant_bands ? 2 : 1;
    auto as = [&](CnChoice::Form f) { return k.form = f, k; };
    if (steps > 1) {
        if (choose_sep_steps(h, t, m, c, k.cn, &k.sc)) return as(CnChoice::separator);
        // no separator plan that fits: the pair form's steps, if the bands are
        // constant (n = 4000, m = 2000, 8 steps: 89 us; cut form 285, sweeps 3499)
        if (h->constant_bands && choose_partition(h, t, m, &k.pc, 3)) return k.cn = 3, as(CnChoice::pair);
    }
    const bool pairs = choose_partition(h, t, m, &k.pc, k.cn);
    if (cut_ok && steps == 1 && choose_cut_cn(h, t, m, k.cn, &k.cc) &&
        takes_cut_cn(h, t, m, pairs ? &k.pc : nullptr, k.cc))
        return as(CnChoice::cut);
    // One step: pentadiagonal, constant bands and a separator shape that fills
    // every CU with whole row runs: the separator kernel's step (coefficients
    // by value).  Hyperdiffusion n = 1024, m = 65536: 234.4 us against 246.2 us
    // in the pair form; for tridiagonal matrices the pair form's step is the
    // faster (periodic diffusion, same size: 221.6 us against 233.5 us).
    if (steps == 1 && h->constant_bands && h->kind == SBS_PENTA && choose_sep(h, t, m, c, &k.sc, 3) &&
        sep_fills(h, t, m, k.sc))
        return as(CnChoice::separator);
    if (pairs) return as(CnChoice::pair);
    // no pair plan that fits: the separator form (pentadiagonal n = 1000 with
    // varying bands, m = 3000: 14 us a step against 128 us), the cut form, or
    // the sweeps
    if (choose_sep_steps(h, t, m, c, k.cn, &k.sc)) return as(CnChoice::separator);
    if (cut_ok && choose_cut_cn(h, t, m, k.cn, &k.cc)) return as(CnChoice::cut);
    return k;
}

// choose_cn, made once for a handle, dtype, m, alignment, one step or several, and
// kept as pick_partition keeps its choices (weighing the shapes takes 5 us).
CnChoice pick_cn(const sbs_lhs *h, int t, int64_t m, const void *c, int steps, bool cut_ok) {
    static std::mutex mu;
    static std::map<std::tuple<uint64_t, int, int64_t, bool, bool, bool>, CnChoice> known;
    const auto key = std::make_tuple(h->id, t, m, aligned(c, 2 * (t == 0 ? 8 : 4)), steps > 1, cut_ok);
    {
        std::lock_guard<std::mutex> g(mu);
        auto it = known.find(key);
        if (it != known.end()) return it->second;
    }
    const CnChoice k = choose_cn(h, t, m, c, steps, cut_ok);
    std::lock_guard<std::mutex> g(mu);
    if (known.size() >= 4096) known.clear();
    try {
        known[key] = k;
    } catch (const std::bad_alloc &) {  // chosen again next time
    }
    return k;
}

// Steps in the cut form, with the unknowns of the cut rows in memory from the
// device's stream-ordered pool for the length of the call.
// False: a graph is being captured (no allocation belongs into it), or there is
// no memory; other forms then run.
bool cut_cn(const sbs_lhs *h, int t, void *c, int64_t m, const CnChoice &k, int steps, hipStream_t s, sbs_status *st) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    void *work = nullptr;
    if (hipStreamIsCapturing(s, &cap) != hipSuccess ||
        (cap == hipStreamCaptureStatusNone && hipMallocAsync(&work, cut_cn_bytes(h, t, m), s) != hipSuccess)) {
        (void)hipGetLastError();  // not this call's error
        return false;
    }
    if (!work) return false;
    const hipError_t e = launch_cut_cn(h, k.cc, t, c, m, k.cn, steps, work, s);
    const hipError_t f = hipFreeAsync(work, s);
    *st = e == hipSuccess && f == hipSuccess ? SBS_OK : SBS_ERR_DEVICE;
    return true;
}

}  // namespace

namespace sbs {

int device_cus(int device) {
    static std::mutex mu;
    static std::map<int, int> known;
    std::lock_guard<std::mutex> g(mu);
    auto it = known.find(device);
    if (it != known.end()) return it->second;
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || cus < 1)
        return 256;  // not kept: asked again next time
    known[device] = cus;
    return cus;
}

int occupancy(const void *fn, int threads, size_t lds) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    static std::mutex mu;
    static std::map<std::tuple<const void *, int, size_t, int>, int> known;
    const auto key = std::make_tuple(fn, threads, lds, dev);
    {
        std::lock_guard<std::mutex> g(mu);
        auto it = known.find(key);
        if (it != known.end()) return it->second;
    }
    int wgs = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&wgs, fn, threads, lds) != hipSuccess) return 0;
    std::lock_guard<std::mutex> g(mu);
    known[key] = wgs;
    return wgs;
}

sbs_status refined_check(const sbs_lhs *h, const float *b, const double *x, int64_t m, int32_t sweeps) {
    if (!h || m < 0 || sweeps < 0 || sweeps > 8 || h->kind == SBS_TRI_PERIODIC) return SBS_ERR_INVALID_ARG;
    if (m == 0) return SBS_OK;
    if (!b || !x || !aligned(b, 8) || !aligned(x, 16)) return SBS_ERR_INVALID_ARG;
    const size_t nb = (size_t)h->n * (size_t)m;
    const char *bx = reinterpret_cast<const char *>(x), *bbp = reinterpret_cast<const char *>(b);
    if (bx < bbp + nb * 4 && bbp < bx + nb * 8) return SBS_ERR_INVALID_ARG;  // b and x overlap
    return SBS_OK;
}

bool refined_fused(const sbs_lhs *h, int64_t m) {
    RefwChoice rc;
    PartChoice pc;
    return choose_refine_wave(h, m, &rc) || choose_partition_refine(h, m, &pc);
}

sbs_status refined_run(const sbs_lhs *h, const float *b, double *x, int64_t m, int32_t sweeps, float *r,
                       hipStream_t s) {
    // Fused paths: one kernel keeps each block of b and x on chip through all
    // passes (needs a partition plan); r is not touched.  First the
    // one-wave-per-block kernel, on overlapping segments of the matrix where two
    // workgroups of it fit on a CU, else on the separator plan, else on longer
    // segments; then the pair form.
    RefwChoice rc;
    // (not where the whole systems are one round of workgroups and the segments
    // two: n = 436, m = 11589 28 against 34 us)
    const int64_t groups = (m + kWave - 1) / kWave, cus = device_cus(h->device);
    const bool halves = h->nseg > 1 && h->segP <= seg_half(h->kind) && (!h->seg_small || m <= 32 * cus) &&
                        (groups > cus || groups * h->nseg <= 2 * cus);
    if (!halves && choose_refine_wave(h, m, &rc))
        return launch_refine_wave(h, rc, b, x, m, sweeps, s) == hipSuccess ? SBS_OK : SBS_ERR_DEVICE;
    if (h->nseg > 0) return launch_refine_segs(h, b, x, m, sweeps, s) == hipSuccess ? SBS_OK : SBS_ERR_DEVICE;
    PartChoice pc;
    if (choose_partition_refine(h, m, &pc))
        return launch_partition_refine(h, pc, b, x, m, sweeps, s) == hipSuccess ? SBS_OK : SBS_ERR_DEVICE;
    // x0 = FP32 solve of b, written as FP64.  r is written in full by the
    // first residual pass before anything reads it.
    hipError_t e = launch_sweep(h, SBS_VARIANT_AUTO, 1, 1, 0, b, x, m, s);
    for (int k = 0; k < sweeps && e == hipSuccess; ++k) {
        // r = fl32(b - A x)   (on later passes fused with x += delta)
        e = launch_refine_step(h, k == 0 ? 0 : 1, b, x, r, r, m, s);
        if (e == hipSuccess) e = launch_sweep(h, SBS_VARIANT_AUTO, 1, 1, 1, r, r, m, s);  // delta
    }
    if (e == hipSuccess && sweeps > 0) e = launch_refine_step(h, 2, b, x, r, nullptr, m, s);  // x += delta
    return e == hipSuccess ? SBS_OK : SBS_ERR_DEVICE;
}

}  // namespace sbs

extern "C" {

const char *sbs_status_str(sbs_status s) {
    switch (s) {
        case SBS_OK: return "ok";
        case SBS_ERR_INVALID_ARG: return "invalid argument";
        case SBS_ERR_ZERO_PIVOT: return "zero or non-finite pivot";
        case SBS_ERR_NONFINITE: return "non-finite matrix coefficient";
        case SBS_ERR_DEVICE: return "device error";
        case SBS_ERR_NO_MEMORY: return "out of memory";
        case SBS_ERR_BUDGET: return "request exceeds the memory budget";
        case SBS_ERR_NOT_FOUND: return "not found";
        case SBS_ERR_TIMEOUT: return "timed out";
        case SBS_ERR_SHUTDOWN: return "server shutting down";
    }
    return "unknown status";
}

const char *sbs_version(void) { return "sbs 0.1 (gfx950)"; }

sbs_status sbs_factor_shared_lhs(int32_t kind, int64_t n, const double *bands, sbs_handle *out,
                                 int64_t *bad_row) {
    int64_t bad = -1;
    if (bad_row) *bad_row = -1;
    if (out) *out = nullptr;
    if (!out || !bands || n < 1 || (kind != SBS_TRI && kind != SBS_PENTA && kind != SBS_TRI_PERIODIC))
        return SBS_ERR_INVALID_ARG;
    // the kernels index rows with 32-bit integers
    if (n > (int64_t)INT32_MAX || (kind == SBS_TRI_PERIODIC && n < 3)) return SBS_ERR_INVALID_ARG;
    for (int64_t i = 0; i < n; ++i)
        for (int k = 0; k < nbands(kind); ++k)
            if (!std::isfinite(entry(bands, kind, n, k, i))) {
                if (bad_row) *bad_row = i;
                return SBS_ERR_NONFINITE;
            }
    sbs_lhs *h = new (std::nothrow) sbs_lhs();
    if (!h) return SBS_ERR_NO_MEMORY;
    static std::atomic<uint64_t> next_id{1};
    h->id = next_id++;
    h->kind = kind;
    h->n = n;
    h->rows = (n + kRowPad - 1) / kRowPad * kRowPad;
    sbs_status st;
    try {
        auto cf = [&](int k, int64_t i) { return entry(bands, kind, n, k, i); };
        if (kind == SBS_TRI) {
            std::vector<TriRow<double>> r(n);
            st = factor_tri_rows(n, cf, r.data(), &bad) ? SBS_OK : SBS_ERR_ZERO_PIVOT;
            if (st == SBS_OK) st = upload<TriRow<double>, TriRow<float>>(h, r, bands);
        } else if (kind == SBS_PENTA) {
            std::vector<PentaRow<double>> r(n);
            st = factor_penta_rows(n, cf, r.data(), &bad) ? SBS_OK : SBS_ERR_ZERO_PIVOT;
            if (st == SBS_OK) st = upload<PentaRow<double>, PentaRow<float>>(h, r, bands);
        } else {
            std::vector<PeriodicRow<double>> r(n);
            st = factor_periodic_rows(n, cf, r.data(), &bad) ? SBS_OK : SBS_ERR_ZERO_PIVOT;
            if (st == SBS_OK) st = upload<PeriodicRow<double>, PeriodicRow<float>>(h, r, bands);
        }
        if (st == SBS_OK) st = build_partitions(h, bands);
        h->constant_bands = constant_bands(bands, kind, n, &h->coef);
    } catch (const std::bad_alloc &) {
        st = SBS_ERR_NO_MEMORY;
    }
    if (st != SBS_OK) {
        if (bad_row) *bad_row = bad;
        sbs_release(h);
        return st;
    }
    *out = h;
    return SBS_OK;
}

sbs_status sbs_factor_uniform(int32_t kind, int64_t n, const double *coeffs, sbs_handle *out, int64_t *bad_row) {
    if (bad_row) *bad_row = -1;
    if (out) *out = nullptr;
    if (!out || !coeffs || n < 1 || n > (int64_t)INT32_MAX) return SBS_ERR_INVALID_ARG;
    if (kind != SBS_TRI && kind != SBS_PENTA && kind != SBS_TRI_PERIODIC) return SBS_ERR_INVALID_ARG;
    const int nb = nbands(kind);
    std::vector<double> bands;
    try {
        bands.resize((size_t)nb * n);
    } catch (const std::bad_alloc &) {
        return SBS_ERR_NO_MEMORY;
    }
    for (int k = 0; k < nb; ++k)
        for (int64_t i = 0; i < n; ++i) bands[(size_t)k * n + i] = coeffs[k];
    return sbs_factor_shared_lhs(kind, n, bands.data(), out, bad_row);
}

sbs_status sbs_release(sbs_handle h) {
    if (!h) return SBS_OK;
    sbs_status st = SBS_OK;
    if (h->dev && hipFree(h->dev) != hipSuccess) st = SBS_ERR_DEVICE;
    if (h->pdev && hipFree(h->pdev) != hipSuccess) st = SBS_ERR_DEVICE;
    delete h;
    return st;
}

sbs_status sbs_handle_info(sbs_handle h, int32_t *kind, int64_t *n, int64_t *device_bytes) {
    if (!h) return SBS_ERR_INVALID_ARG;
    if (kind) *kind = h->kind;
    if (n) *n = h->n;
    if (device_bytes) *device_bytes = h->device_bytes;
    return SBS_OK;
}

sbs_status sbs_solve_batch_variant(sbs_handle h, void *rhs, int64_t m, int32_t dtype, int32_t variant,
                                   void *stream) {
    if (!h || m < 0 || (dtype != SBS_F64 && dtype != SBS_F32)) return SBS_ERR_INVALID_ARG;
    if (variant < SBS_VARIANT_AUTO || variant > SBS_VARIANT_PARTITION) return SBS_ERR_INVALID_ARG;
    if (variant == SBS_VARIANT_RESIDENT && h->n > 64) return SBS_ERR_INVALID_ARG;
    if (m == 0) return SBS_OK;
    if (!rhs || !aligned(rhs, dtype == SBS_F64 ? 8 : 4)) return SBS_ERR_INVALID_ARG;
    if (m > (int64_t)0x7fffffff * kWave) return SBS_ERR_INVALID_ARG;
    if (variant == SBS_VARIANT_CHUNKED && chunked_lds_bytes(h, dtype == SBS_F64 ? 0 : 1) > kMaxLdsBytes)
        return SBS_ERR_INVALID_ARG;
    const int t = dtype == SBS_F64 ? 0 : 1;
    hipError_t e;
    if (variant == SBS_VARIANT_AUTO || variant == SBS_VARIANT_PARTITION) {
        SepChoice sc;
        PartChoice pc;
        CutChoice cut;
        const int form = pick_partition(h, t, m, rhs, variant == SBS_VARIANT_AUTO, &sc, &pc, &cut);
        hipStream_t s = static_cast<hipStream_t>(stream);
        if (cut.S)
            e = launch_cut(h, cut, t, rhs, m, s);
        else if (form == 1)
            e = launch_sep(h, sc, t, rhs, m, s);
        else if (form == 2)
            e = launch_partition(h, pc, t, t, t, rhs, rhs, m, s);
        else if (variant == SBS_VARIANT_PARTITION)
            return SBS_ERR_INVALID_ARG;
        else
            e = launch_sweep(h, variant, t, t, t, rhs, rhs, m, s);
        return e == hipSuccess ? SBS_OK : SBS_ERR_DEVICE;
    }
    e = launch_sweep(h, variant, t, t, t, rhs, rhs, m, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? SBS_OK : SBS_ERR_DEVICE;
}

sbs_status sbs_solve_batch_partition(sbs_handle h, void *rhs, int64_t m, int32_t dtype, int32_t form, int32_t lb,
                                     int32_t vec, int32_t S, int32_t flags, void *stream) {
    if (!h || m < 0 || (dtype != SBS_F64 && dtype != SBS_F32) || (form != 0 && form != 1)) return SBS_ERR_INVALID_ARG;
    if (m == 0) return SBS_OK;
    if (!rhs || !aligned(rhs, dtype == SBS_F64 ? 8 : 4) || m > (int64_t)0x7fffffff * kWave) return SBS_ERR_INVALID_ARG;
    const int t = dtype == SBS_F64 ? 0 : 1;
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipError_t e;
    if (form == 1) {
        SepChoice sc;
        if (flags < 0 || flags > 0xffff || !sep_shape(h, t, m, rhs, lb, vec, S, flags, &sc)) return SBS_ERR_INVALID_ARG;
        e = launch_sep(h, sc, t, rhs, m, s);
    } else {
        PartChoice pc;
        if (vec != 1 || flags != 0 || !part_shape(h, t, m, lb, S, &pc)) return SBS_ERR_INVALID_ARG;
        e = launch_partition(h, pc, t, t, t, rhs, rhs, m, s);
    }
    return e == hipSuccess ? SBS_OK : SBS_ERR_DEVICE;
}

sbs_status sbs_partition_shape(sbs_handle h, int64_t m, int32_t dtype, const void *rhs, int32_t *form, int32_t *lb,
                               int32_t *vec, int32_t *S) {
    if (!h || m < 1 || (dtype != SBS_F64 && dtype != SBS_F32) || !form || !lb || !vec || !S)
        return SBS_ERR_INVALID_ARG;
    const int t = dtype == SBS_F64 ? 0 : 1;
    SepChoice sc;
    PartChoice pc;
    const int pick = pick_partition(h, t, m, rhs, true, &sc, &pc);
    if (pick == 1) {
        *form = 1;
        *lb = h->sep[sc.plan].lb;
        *vec = sc.vec;
        *S = sc.S;
    } else if (pick == 2) {
        *form = 0;
        *lb = h->part[pc.plan].lb;
        *vec = 1;
        *S = pc.S;
    } else {
        *form = *lb = *vec = *S = 0;
        return SBS_ERR_NOT_FOUND;
    }
    return SBS_OK;
}

sbs_status sbs_auto_variant(sbs_handle h, int64_t m, int32_t dtype, int32_t *variant) {
    if (!h || !variant || m < 1 || (dtype != SBS_F64 && dtype != SBS_F32)) return SBS_ERR_INVALID_ARG;
    const int t = dtype == SBS_F64 ? 0 : 1;
    PartChoice pc;
    SepChoice sc;
    // (shapes for right-hand sides aligned to 16 bytes)
    *variant = pick_partition(h, t, m, nullptr, true, &sc, &pc) ? SBS_VARIANT_PARTITION : choose_variant(h, t);
    return SBS_OK;
}

sbs_status sbs_solve_batch(sbs_handle h, void *rhs, int64_t m, int32_t dtype, void *stream) {
    return sbs_solve_batch_variant(h, rhs, m, dtype, SBS_VARIANT_AUTO, stream);
}

size_t sbs_refined_workspace_bytes(sbs_handle h, int64_t m) {
    if (!h || m < 0) return 0;
    // One FP32 residual / correction array of n*m, rounded to 256 bytes.
    return ((size_t)h->n * (size_t)m * sizeof(float) + 255) / 256 * 256;
}

sbs_status sbs_solve_batch_refined(sbs_handle h, const float *b, double *x, int64_t m, int32_t sweeps, void *work,
                                   size_t work_bytes, void *stream) {
    const sbs_status st = refined_check(h, b, x, m, sweeps);
    if (st != SBS_OK || m == 0) return st;
    if (!work || work_bytes < sbs_refined_workspace_bytes(h, m) || !aligned(work, 8)) return SBS_ERR_INVALID_ARG;
    return refined_run(h, b, x, m, sweeps, static_cast<float *>(work), static_cast<hipStream_t>(stream));
}

sbs_status sbs_cn_step(sbs_handle h, void *c, int64_t m, int32_t dtype, int32_t steps, void *stream) {
    if (!h || m < 0 || steps < 0 || (dtype != SBS_F64 && dtype != SBS_F32)) return SBS_ERR_INVALID_ARG;
    if (m == 0 || steps == 0) return SBS_OK;
    if (!c || !aligned(c, dtype == SBS_F64 ? 8 : 4)) return SBS_ERR_INVALID_ARG;
    if (m > (int64_t)0x7fffffff * kWave) return SBS_ERR_INVALID_ARG;
    const int t = dtype == SBS_F64 ? 0 : 1;
    hipStream_t s = static_cast<hipStream_t>(stream);
    CnChoice k = pick_cn(h, t, m, c, steps, true);
    if (k.form == CnChoice::cut) {
        sbs_status st = SBS_OK;
        if (cut_cn(h, t, c, m, k, steps, s, &st)) return st;
        k = pick_cn(h, t, m, c, steps, false);
    }
    hipError_t e = hipSuccess;
    if (k.form == CnChoice::separator)
        e = launch_sep(h, k.sc, t, c, m, s, steps);
    else if (k.form == CnChoice::pair && k.cn == 3)
        e = launch_partition(h, k.pc, t, t, t, c, c, m, s, 3, steps);
    else
        for (int q = 0; q < steps && e == hipSuccess; ++q)
            e = k.form == CnChoice::pair ? launch_partition(h, k.pc, t, t, t, c, c, m, s, k.cn) : launch_cn(h, t, c, m, s);
    return e == hipSuccess ? SBS_OK : SBS_ERR_DEVICE;
}

sbs_status sbs_auto_cut(sbs_handle h, int64_t m, int32_t dtype, const void *rhs, int32_t cn_steps, int32_t *segments,
                        int32_t *S) {
    if (!h || m < 1 || cn_steps < 0 || (dtype != SBS_F64 && dtype != SBS_F32) || !segments || !S)
        return SBS_ERR_INVALID_ARG;
    const int t = dtype == SBS_F64 ? 0 : 1;
    CutChoice cut;
    if (cn_steps) {
        const CnChoice k = pick_cn(h, t, m, rhs, cn_steps, true);
        if (k.form == CnChoice::cut) cut = k.cc;
    } else {
        SepChoice sc;
        PartChoice pc;
        pick_partition(h, t, m, rhs, true, &sc, &pc, &cut);
    }
    *segments = cut.S ? h->cut.Q : 0;
    *S = cut.S;
    return SBS_OK;
}

sbs_status sbs_transpose(const void *src, void *dst, int64_t rows, int64_t cols, int32_t dtype, void *stream) {
    if (rows < 0 || cols < 0 || (dtype != SBS_F64 && dtype != SBS_F32)) return SBS_ERR_INVALID_ARG;
    if (rows == 0 || cols == 0) return SBS_OK;
    if (!src || !dst) return SBS_ERR_INVALID_ARG;
    const size_t eb = dtype == SBS_F64 ? 8 : 4;
    const size_t bytes = (size_t)rows * (size_t)cols * eb;
    const char *s = static_cast<const char *>(src), *d = static_cast<const char *>(dst);
    if (s < d + bytes && d < s + bytes) return SBS_ERR_INVALID_ARG;
    if (!aligned(src, eb) || !aligned(dst, eb)) return SBS_ERR_INVALID_ARG;
    hipError_t e = launch_transpose(src, dst, rows, cols, (int)eb, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? SBS_OK : SBS_ERR_DEVICE;
}

sbs_status sbs_adi_step(sbs_handle hy, sbs_handle hx, double *grid, double *work, int64_t ny, int64_t nx,
                        void *stream) {
    if (!hy || !hx || ny < 1 || nx < 1 || hy->n != ny || hx->n != nx) return SBS_ERR_INVALID_ARG;
    if (!grid || !work) return SBS_ERR_INVALID_ARG;
    sbs_status st = sbs_solve_batch(hy, grid, nx, SBS_F64, stream);          // along y
    if (st != SBS_OK) return st;
    // Along x the systems are the grid's rows.  With a partition plan they
    // are solved where they are (each lane reads its block of a row as one
    // contiguous run); otherwise through the interleaved layout of the
    // transpose.
    PartChoice pc;
    if (choose_partition(hx, 0, ny, &pc, false, true))
        return launch_partition_rows(hx, pc, grid, ny, static_cast<hipStream_t>(stream)) == hipSuccess
                   ? SBS_OK
                   : SBS_ERR_DEVICE;
    st = sbs_transpose(grid, work, ny, nx, SBS_F64, stream);                   // (ny, nx) -> (nx, ny)
    if (st == SBS_OK) st = sbs_solve_batch(hx, work, ny, SBS_F64, stream);      // along x
    if (st == SBS_OK) st = sbs_transpose(work, grid, nx, ny, SBS_F64, stream);  // back
    return st;
}

}  // extern "C"
