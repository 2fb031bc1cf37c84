// Separator-partitioned solve (several lanes per system) for plain solves of
// interleaved right-hand sides.
//
// The rows of every system are cut into P blocks of LB rows.  The last H rows
// of each block (but the last, unless the matrix is periodic) are separator
// rows; the others are interior rows.  A workgroup holds S systems x P
// blocks: lane (p, s) loads rows [p*LB, (p+1)*LB) of VEC adjacent systems
// (VEC = 2: one 16-byte access per FP64 row), and then, per group of S
// systems:
//   1. runs the Section 3.1 / 4.1 recurrences over its block with the
//      block's interior factor (separator rows are identity rows, so they pass
//      through holding their right-hand sides);
//   2. writes to LDS its two parts of the separator right-hand sides
//      yhat = f_sep - (couplings of the separator rows to the interior rows
//      on either side) . g: its own separator's f_sep less the couplings to
//      the block's last interior rows (redL), and minus the previous
//      separator's couplings to the block's first rows (redR); one barrier;
//   3. the separators of all S systems follow as Z = S^{-1} Yhat, a dense
//      (Nr x Nr)(Nr x S) product on the matrix cores in FP64 (per-lane dot
//      products otherwise);
//   4. corrects its interior rows x = g - V z_own - W z_prev, takes its
//      separator rows from z, and stores every row once, non-temporally,
//      loading the next group's rows into the registers it frees.
// Each right-hand side crosses HBM once in and once out (16 bytes per FP64
// unknown).  The block factors, spikes V / W, separator band rows and S^{-1}
// depend only on the shared matrix; they are computed once on the host and
// copied into LDS once per persistent workgroup (where the whole plan does
// not fit, only S^{-1} is, and the rest is read from global memory).
#include <algorithm>
#include <type_traits>

#include "internal.h"

namespace sbs {
namespace {

// (a pair is one 16- or 8-byte access wherever it starts: rows of an odd
// number of systems start at odd elements, and global accesses of gfx950 need
// the alignment of a 4-byte word only)
typedef double D2 __attribute__((ext_vector_type(2), aligned(8)));
typedef float F2 __attribute__((ext_vector_type(2), aligned(4)));
typedef double D4 __attribute__((ext_vector_type(4)));

template <int KIND, typename T>
struct RowOf;
template <typename T>
struct RowOf<SBS_TRI, T> {
    using type = TriRow<T>;
};
template <typename T>
struct RowOf<SBS_PENTA, T> {
    using type = PentaRow<T>;
};

template <typename T>
struct Pair;
template <>
struct Pair<double> {
    using type = D2;
};
template <>
struct Pair<float> {
    using type = F2;
};

// VEC adjacent values of one row (one 8/16-byte access for VEC = 2).
template <typename T, int VEC>
__device__ __forceinline__ void load_vec(const T *p, T (&v)[VEC]) {
    if constexpr (VEC == 1) {
        v[0] = *p;
    } else {
        const typename Pair<T>::type a = *reinterpret_cast<const typename Pair<T>::type *>(p);
        v[0] = a.x;
        v[1] = a.y;
    }
}

template <typename T, int VEC>
__device__ __forceinline__ void store_vec_nt(T *p, const T (&v)[VEC]) {
    if constexpr (VEC == 1) {
        __builtin_nontemporal_store(v[0], p);
    } else {
        typename Pair<T>::type a;
        a.x = v[0];
        a.y = v[1];
        __builtin_nontemporal_store(a, reinterpret_cast<typename Pair<T>::type *>(p));
    }
}

__device__ __forceinline__ int align16(int b) { return (b + 15) / 16 * 16; }

// Copies the plan blob into LDS, eight 16-byte loads in flight per thread.
__device__ __forceinline__ void stage(unsigned char *lds, const unsigned char *blob, int bytes) {
    typedef unsigned int U4 __attribute__((ext_vector_type(4)));
    constexpr int U = 8;
    const U4 *src = reinterpret_cast<const U4 *>(blob);
    U4 *dst = reinterpret_cast<U4 *>(lds);
    const int total = bytes / 16, step = blockDim.x;
    int i = threadIdx.x;
    for (; i + (U - 1) * step < total; i += U * step) {
        U4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = src[i + u * step];
#pragma unroll
        for (int u = 0; u < U; ++u) dst[i + u * step] = v[u];
    }
    for (; i < total; i += step) dst[i] = src[i];
}

struct SepArgs {
    int fac_bytes, spk_bytes, scf_bytes, sinv_bytes, map_bytes;
    int n, P, Nr, S, ngroups, periodic, flags;
    int kofs, kw;  // window of the S^{-1} product (kw = 0: every column)
    int64_t m;
    BandCoef coef;  // Crank-Nicolson steps: the matrix's constant band values
};
// And those of the kernels for several steps, band rows and the cut form only: the
// arguments a plain solve does not read make its launch longer (see k_sep).
struct SepMoreArgs : SepArgs {
    int steps;             // Crank-Nicolson steps to run
    const BandRow *bands;  // the matrix's band rows
    const CutSeg *segs;  // the cut form: Q segments
    int Q, per, per_last;  // and the workgroups of each, and of the last
    const void *ucut;      // its Crank-Nicolson steps: the unknowns of the cut rows, [cut][H][m]
};

// Device memory that does not change while a kernel runs: uniform reads
// become scalar loads.
template <typename T>
using cptr = const __attribute__((address_space(4))) T *;

// Z = S^{-1} Yhat for the group on the matrix cores (Yhat = redl + redr, the
// two parts of the separator right-hand sides): 16 x 16 output tiles of
// v_mfma_f64_16x16x4f64 shared out over the waves (lane l holds
// A[l % 16][l / 16] and B[l / 16][l % 16]; item r of the result is
// D[4 r + l / 16][l % 16]).  Column s of Yhat / Z is at red / z + s * ldr.
//
// One 16 x 16 tile of Z: the lane's row i of S^{-1} and column j of Yhat
// over columns kb .. kb + kn - 1, four per matrix-core step.  Every operand
// is read at an index clamped inside the buffers, so that no read is
// conditional (as branches around each read the steps ran one after
// another), and the next step's operands are read before the current step's
// product.  Rows i >= Nr and columns j >= S of the tile hold other rows' and
// columns' values and are never stored; entries of S^{-1} past column Nr - 1
// are multiplied by 0 (finite values: the entries of S^{-1}), so the
// right-hand sides read there add nothing.
__device__ __forceinline__ D4 sep_tile(const double *sinv, const double *redl, const double *redr, int Nr, int S,
                                       int ldr, int i, int j, int lk, int kb, int kn) {
    const double *arow = sinv + (size_t)min(i, Nr - 1) * Nr;
    const double *bl = redl + min(j, S - 1) * ldr, *br = redr + min(j, S - 1) * ldr;
    auto opnd = [&](int k0, double &a, double &b) {
        const int k = k0 + lk, kc = min(k, Nr - 1);
        a = arow[kc] * (k < Nr ? 1.0 : 0.0);
        b = bl[kc] + br[kc];
    };
    D4 acc = {0.0, 0.0, 0.0, 0.0};
    double a, b;
    opnd(kb, a, b);
    for (int k0 = kb + 4; k0 < kb + kn; k0 += 4) {
        double an, bn;
        opnd(k0, an, bn);
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 0);
        a = an;
        b = bn;
    }
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 0);
}

// The entries of S^{-1} outside a tile's window are 0 (the plan drops
// entries below 2^-60 / Nr of their row's largest), so the tile reads only
// columns k0 .. k0 + kw - 1, k0 = min(max(i0 + kofs, 0), max(Nr4 - kw, 0)),
// and the result is the product over every column bit for bit (the skipped
// terms are exact zeros); kw = 0 reads every column.
//
// ALIAS: z is redl's storage (the LDS holds no third buffer); each wave has
// at most one tile, and writes it only after every wave has read Yhat.
template <bool ALIAS>
__device__ __forceinline__ void sep_mma(const double *sinv, const double *redl, const double *redr, double *z, int Nr,
                                        int S, int ldr, int kofs, int kw) {
    // the thread's coordinates, made opaque at each call: the tile addresses
    // below are formed per call rather than kept live across the group loop
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave), nwaves = blockDim.x / kWave;
    const int mt = (Nr + 15) / 16, ntiles = mt * ((S + 15) / 16);
    const int lr = lane % 16, lk = lane / 16;
    const int Nr4 = (Nr + 3) / 4 * 4, kn = kw ? kw : Nr;
    auto kfirst = [&](int i0) { return kw ? min(max(i0 + kofs, 0), max(Nr4 - kw, 0)) : 0; };
    if constexpr (ALIAS) {
        const bool have = wave < ntiles;
        const int i0 = (wave % mt) * 16, j0 = (wave / mt) * 16;
        const int i = i0 + lr, j = j0 + lr;
        D4 acc = {0.0, 0.0, 0.0, 0.0};
        if (have) acc = sep_tile(sinv, redl, redr, Nr, S, ldr, i, j, lk, kfirst(i0), kn);
        __syncthreads();
        if (have) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = i0 + 4 * r + lk;
                if (row < Nr && j < S) z[j * ldr + row] = acc[r];
            }
        }
        return;
    }
    for (int tile = wave; tile < ntiles; tile += nwaves) {
        const int i0 = (tile % mt) * 16, j0 = (tile / mt) * 16;
        const int i = i0 + lr, j = j0 + lr;
        const D4 acc = sep_tile(sinv, redl, redr, Nr, S, ldr, i, j, lk, kfirst(i0), kn);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = i0 + 4 * r + lk;
            if (row < Nr && j < S) z[j * ldr + row] = acc[r];
        }
    }
}

// LDS layout after the blob: the two parts of the separator right-hand
// sides, redL and redR [S][ldr], and (FP64) the separators z [S][ldr].
template <typename T>
__host__ __device__ __forceinline__ int sep_red_bytes(int S, int Nr) {
    return (S * (Nr + 1) * (int)sizeof(T) + 15) / 16 * 16;
}

// Compiler-only fence: `v` must be computed here, and no memory access moves
// across (emits no instruction).  Keeps the coefficient reads of later rows
// from being hoisted to the start of a loop, where they would hold every
// row's coefficients in registers at once.
template <typename T>
__device__ __forceinline__ void pin(T &v) {
    asm volatile("" : "+v"(v) : : "memory");
}

constexpr int G = 4;  // rows per coefficient group (2 where registers are short)

// The block's forward and backward sweeps (Sections 3.1 / 4.1) over VEC
// systems in registers, with the block's factor rows from LDS.
// OPQ (rows in global memory): the row pointer is made opaque before each
// group of rows is read, so that the read-only loads are not all hoisted to
// the start (the fences below do not hold back loads of memory that nothing
// in the kernel writes).
template <int KIND, typename T, int LB, int VEC, bool OPQ>
__device__ __forceinline__ void block_sweeps(const typename RowOf<KIND, T>::type *fr, T (&x)[LB][VEC]) {
    // coefficient rows per group: fewer when the block's values fill the registers
    constexpr int NG = LB / G;
    if constexpr (KIND == SBS_TRI) {
        T cf[2][G][2];
        T y1[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) y1[v] = T(0);
        if constexpr (OPQ) asm volatile("" : "+v"(fr));
#pragma unroll
        for (int u = 0; u < G; ++u) cf[0][u][0] = fr[u].a_s, cf[0][u][1] = fr[u].inv;
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            if (g + 1 < NG) {
                if constexpr (OPQ) asm volatile("" : "+v"(fr));
#pragma unroll
                for (int u = 0; u < G; ++u)
                    cf[(g + 1) & 1][u][0] = fr[(g + 1) * G + u].a_s, cf[(g + 1) & 1][u][1] = fr[(g + 1) * G + u].inv;
            }
#pragma unroll
            for (int u = 0; u < G; ++u)
#pragma unroll
                for (int v = 0; v < VEC; ++v)  // y_i = d_i / den_i - (a_i / den_i) y_{i-1}
                    y1[v] = x[g * G + u][v] = fma(-cf[g & 1][u][0], y1[v], x[g * G + u][v] * cf[g & 1][u][1]);
            pin(y1[0]);
        }
        T ch[2][G];
        T x1[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) x1[v] = T(0);
        if constexpr (OPQ) asm volatile("" : "+v"(fr));
#pragma unroll
        for (int u = 0; u < G; ++u) ch[(NG - 1) & 1][u] = fr[LB - 1 - u].chat;
#pragma unroll
        for (int g = NG - 1; g >= 0; --g) {
            if (g > 0) {
                if constexpr (OPQ) asm volatile("" : "+v"(fr));
#pragma unroll
                for (int u = 0; u < G; ++u) ch[(g - 1) & 1][u] = fr[g * G - 1 - u].chat;
            }
#pragma unroll
            for (int u = 0; u < G; ++u) {
                const int t = g * G + G - 1 - u;
#pragma unroll
                for (int v = 0; v < VEC; ++v)  // x_i = y_i - chat_i x_{i+1}
                    x1[v] = x[t][v] = fma(-ch[g & 1][u], x1[v], x[t][v]);
            }
            pin(x1[0]);
        }
    } else {
        T cf[2][G][3];
        T g1[VEC], g2[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) g1[v] = g2[v] = T(0);
        if constexpr (OPQ) asm volatile("" : "+v"(fr));
#pragma unroll
        for (int u = 0; u < G; ++u) cf[0][u][0] = fr[u].eps_s, cf[0][u][1] = fr[u].beta_s, cf[0][u][2] = fr[u].inv;
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            if (g + 1 < NG) {
                if constexpr (OPQ) asm volatile("" : "+v"(fr));
#pragma unroll
                for (int u = 0; u < G; ++u) {
                    const int t = (g + 1) * G + u;
                    cf[(g + 1) & 1][u][0] = fr[t].eps_s;
                    cf[(g + 1) & 1][u][1] = fr[t].beta_s;
                    cf[(g + 1) & 1][u][2] = fr[t].inv;
                }
            }
#pragma unroll
            for (int u = 0; u < G; ++u)
#pragma unroll
                for (int v = 0; v < VEC; ++v) {  // g_i = (f_i - eps_i g_{i-2} - beta_i g_{i-1}) / alpha_i
                    const T *c = cf[g & 1][u];
                    const T gg = fma(-c[1], g1[v], fma(-c[0], g2[v], x[g * G + u][v] * c[2]));
                    g2[v] = g1[v];
                    g1[v] = gg;
                    x[g * G + u][v] = gg;
                }
            pin(g1[0]);
        }
        T cb[2][G][2];
        T x1[VEC], x2[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) x1[v] = x2[v] = T(0);
        if constexpr (OPQ) asm volatile("" : "+v"(fr));
#pragma unroll
        for (int u = 0; u < G; ++u) cb[(NG - 1) & 1][u][0] = fr[LB - 1 - u].gamma, cb[(NG - 1) & 1][u][1] = fr[LB - 1 - u].delta;
#pragma unroll
        for (int g = NG - 1; g >= 0; --g) {
            if (g > 0) {
                if constexpr (OPQ) asm volatile("" : "+v"(fr));
#pragma unroll
                for (int u = 0; u < G; ++u) {
                    const int t = g * G - 1 - u;
                    cb[(g - 1) & 1][u][0] = fr[t].gamma;
                    cb[(g - 1) & 1][u][1] = fr[t].delta;
                }
            }
#pragma unroll
            for (int u = 0; u < G; ++u) {
                const int t = g * G + G - 1 - u;
#pragma unroll
                for (int v = 0; v < VEC; ++v) {  // x_i = g_i - gamma_i x_{i+1} - delta_i x_{i+2}
                    const T xx = fma(-cb[g & 1][u][0], x1[v], fma(-cb[g & 1][u][1], x2[v], x[t][v]));
                    x2[v] = x1[v];
                    x1[v] = xx;
                    x[t][v] = xx;
                }
            }
            pin(x1[0]);
        }
    }
}

// flags: bit 0 XCD-grouped order of the groups (the workgroups a chiplet
// runs at once take adjacent groups); bit 2 workgroups start out of step (see
// below); bit 6 the S^{-1} product over every column instead of the plan's
// window (same result).  (Issuing the next group's loads into registers while the current
// group is stored was measured slower: each wave's loads then queue behind
// its stores.)
//
// GF: the plan does not fit the LDS with the group's buffers; only S^{-1}
// is copied there, and the factor rows, spikes, separator rows and block map
// are read from global memory (the caches hold them: every group reads the
// same plan).  The separators then overwrite redL, and the corrected rows
// are stored after all of them are computed (a spike load issued after a
// store would wait for that store).
//
// CN: a.steps Crank-Nicolson steps c <- A^{-1} (2I - A) c (Sections 3.2, 4.2):
// with u = A^{-1} c in registers, row t of the output is
// 2 u_t - sum_e coef_e u_{t-H+e}, with the row's own coefficients (CN 1: the
// band rows a.bands, staged in LDS) or those of a matrix whose bands are
// constant (CN 2 and 3: the values in a.coef).  The rows
// above the block are the previous block's separators (known to the lane);
// the first H rows of the next block come through LDS, one more barrier.
// Values outside the matrix are 0, so the constant coefficients also give
// the truncated rows at its ends.  The group's systems are whole in the
// workgroup, so every step but the last leaves its rows in the registers
// for the next one: HBM is crossed once in and once out however many steps a
// call asks for, and a step costs its arithmetic and barriers only.  CN 3 is
// one step, with each row stored as it is formed: fewer values live, and the
// stores spread out (hyperdiffusion n = 600, m = 100000: 234 us, through the
// several steps' kernel 277 us).
// (Hyperdiffusion n = 1024, m = 65536, 8 steps per call: 597 us, with one
// launch and one pass over HBM per step 1827 us; periodic diffusion n = 512,
// m = 6000, 20 steps: 89 us against 332 us.)  The rows are stored after the
// last step, not as they are formed: with the pairs of an odd batch as a
// branch in the output loop 66 registers spilled.
// With SEG one step per launch; the unknowns of the cut rows are in ucut, and
// the workgroup before a cut also steps its rows.
//
// SEG: the cut form.  A workgroup solves one segment of the matrix as one of
// its own (its plan, its rows), after k_cut_rows has put the unknowns of the
// cut rows into the array: the segment's first and last H right-hand sides
// lose their couplings to them.  A segment of 256 rows leaves room for 128
// systems per workgroup, whatever n is.
// m may be odd: a lane at or past the last system takes the last two and
// stores the last one only, since the other may be another workgroup's.
template <int KIND, typename T, int LB, int VEC, int MAXT, bool GF, int CN = 0, bool SEG = false>
__global__ __launch_bounds__(MAXT) void k_sep(const unsigned char *__restrict__ blob,
                                              std::conditional_t<SEG || CN == 1 || CN == 2, SepMoreArgs, SepArgs> a,
                                              const T *in, T *out) {
    using Row = typename RowOf<KIND, T>::type;
    constexpr int H = KIND / 2, NB = 2 * H + 1, NI = LB - H;
    constexpr bool MMA = sizeof(T) == 8;
    extern __shared__ __align__(16) unsigned char lds[];
    bool cut_lo = false, cut_hi = false;
    int lo_at = 0, lo_cut = 0, hi_cut = 0, seg_b = 0, seg_grid = 1;
    T clo[H][H], chi[H][H];
    if constexpr (SEG) {
        constexpr int tc = sizeof(T) == 8 ? 0 : 1;
        // the segments in turn, then what the last one has fewer or more
        const int each = min(a.per, a.per_last), rest = (int)blockIdx.x - a.Q * each;
        int k;
        if (rest < 0) {
            k = blockIdx.x % a.Q;
            seg_b = blockIdx.x / a.Q;
        } else if (a.per > each) {
            k = rest % (a.Q - 1);
            seg_b = each + rest / (a.Q - 1);
        } else {
            k = a.Q - 1;
            seg_b = each + rest;
        }
        seg_grid = k == a.Q - 1 ? a.per_last : a.per;
        const cptr<CutSeg> s = (cptr<CutSeg>)(a.segs + k);
        blob = s->blob[tc];
        a.fac_bytes = s->fac[tc];
        a.spk_bytes = s->spk[tc];
        a.scf_bytes = s->scf[tc];
        a.sinv_bytes = s->sinv[tc];
        a.map_bytes = s->map;
        a.n = s->rows;
        a.P = s->P;
        a.Nr = s->Nr;
        a.kofs = s->kofs;
        a.kw = s->kw;
        in += (int64_t)s->row0 * a.m;
        out += (int64_t)s->row0 * a.m;
        cut_lo = s->has_lo != 0;
        cut_hi = s->has_hi != 0;
        lo_at = s->lo_at;
        lo_cut = s->lo_cut;
        hi_cut = s->hi_cut;
        if constexpr (CN == 1) a.bands += s->row0;
#pragma unroll
        for (int t = 0; t < H; ++t)
#pragma unroll
            for (int c = 0; c < H; ++c) {
                clo[t][c] = (T)s->lo[t][c];
                chi[t][c] = (T)s->hi[t][c];
            }
    }
    const int P = a.P, Nr = a.Nr, S = a.S, n = a.n;
    const int blob_bytes = a.fac_bytes + a.spk_bytes + a.scf_bytes + a.sinv_bytes + a.map_bytes;
    const int sinv_at = a.fac_bytes + a.spk_bytes + a.scf_bytes;
    const Row *lfac;
    const T *lspk, *lscf, *lsinv;
    const int *lmap;
    if constexpr (GF) {
        lfac = reinterpret_cast<const Row *>(blob);
        lspk = reinterpret_cast<const T *>(blob + a.fac_bytes);
        lscf = reinterpret_cast<const T *>(blob + a.fac_bytes + a.spk_bytes);
        lmap = reinterpret_cast<const int *>(blob + sinv_at + a.sinv_bytes);
        lsinv = reinterpret_cast<const T *>(lds);
    } else {
        lfac = reinterpret_cast<const Row *>(lds);
        lspk = reinterpret_cast<const T *>(lds + a.fac_bytes);
        lscf = reinterpret_cast<const T *>(lds + a.fac_bytes + a.spk_bytes);
        lsinv = reinterpret_cast<const T *>(lds + sinv_at);
        lmap = reinterpret_cast<const int *>(lds + sinv_at + a.sinv_bytes);
    }
    const int plan_lds = GF ? a.sinv_bytes : blob_bytes;
    // odd stride: the systems' columns fall in different banks (two Crank-Nicolson
    // steps of 1024 tridiagonal systems, FP32, n = 2048, 63 separators: at a stride
    // of 64 78 us, of 63 29 us; n = 1024, 31 separators, 28 and 18 us)
    const int ldr = Nr | 1;
    T *lredl = reinterpret_cast<T *>(lds + plan_lds);
    T *lredr = reinterpret_cast<T *>(lds + plan_lds + sep_red_bytes<T>(S, Nr));
    // flags bit 5 (GF only, set by the launch when the LDS has no room for a
    // third buffer): the separators overwrite redL
    const bool alias = GF && (a.flags & 32);
    T *lz = alias ? lredl : reinterpret_cast<T *>(lds + plan_lds + 2 * sep_red_bytes<T>(S, Nr));
    // CN: the first H rows of every block of the group, [S][P][H]
    T *ltop = reinterpret_cast<T *>(lds + plan_lds + (alias ? 2 : 3) * sep_red_bytes<T>(S, Nr));
    // CN 1: the band rows, [P * LB][NB], 0 outside the matrix
    T *lband = reinterpret_cast<T *>(reinterpret_cast<unsigned char *>(ltop) + align16(S * P * H * (int)sizeof(T)));
    if constexpr (CN == 1) {
        for (int i = threadIdx.x; i < P * LB; i += blockDim.x)
#pragma unroll
            for (int e = 0; e < NB; ++e) lband[i * NB + e] = i < n ? (T)a.bands[i].c[e] : T(0);
    }


    const int Ls = S / VEC;  // lanes per block row
    const int l = threadIdx.x, p0 = l / Ls, sl = l - p0 * Ls;
    // lanes past the last block (the workgroup is whole waves) have no rows and
    // no separators: they load and store nothing
    const int p = min(p0, P - 1);
    const bool active = p0 < P;
    const int rows = active ? n : 0;
    const int r0 = p * LB;
    const bool has_sep = active && (a.periodic || p < P - 1), has_prev = active && (a.periodic || p > 0);
    const int pp = p == 0 ? P - 1 : p - 1;
    const int s0 = sl * VEC;  // the lane's first system within the group
    const int64_t m = a.m;
    const bool full = r0 + LB <= rows;
    const int grid = SEG ? seg_grid : gridDim.x;
    int b = SEG ? seg_b : blockIdx.x;
    if ((a.flags & 1) && grid % 8 == 0) b = (b % 8) * (grid / 8) + b / 8;

    T x[LB][VEC];
    // lanes past the last system take the last VEC systems: same values, same
    // addresses, so their duplicate stores are harmless
    auto col = [&](int g) { return min((int64_t)g * S + s0, m - VEC); };
    // (an odd batch: the cut form and Crank-Nicolson steps take pairs all the same)
    constexpr bool ANYM = (SEG || (CN && CN != 3)) && VEC == 2;
    auto last_only = [&](int g) { return ANYM && (int64_t)g * S + s0 > m - VEC; };
    // SEG: the unknowns of the cut rows before the lane's block and after it (a
    // single block has both only if the matrix is periodic, so tridiagonal:
    // pentadiagonal lanes need one of the two and keep it in `before`)
    const bool at_lo = SEG && cut_lo && p0 == 0, at_hi = SEG && cut_hi && p0 == P - 1;
    T before[H][VEC], after[H][VEC];
    auto load_group = [&](int g) {
        const T *src = in + (int64_t)r0 * m + col(g);
        if constexpr (SEG) {
            // (Crank-Nicolson steps leave the cut rows' own values where they are)
            const T *qlo = src + (int64_t)lo_at * m, *qhi = src + (int64_t)(n - r0) * m;
            if constexpr (CN) {
                qlo = static_cast<const T *>(a.ucut) + (int64_t)lo_cut * H * m + col(g);
                qhi = static_cast<const T *>(a.ucut) + (int64_t)hi_cut * H * m + col(g);
            }
            if (H == 1 ? at_lo : at_lo || at_hi) {
                const T *q = at_lo ? qlo : qhi;
#pragma unroll
                for (int c = 0; c < H; ++c) load_vec<T, VEC>(q + (int64_t)c * m, before[c]);
            }
            if constexpr (H == 1)
                if (at_hi) load_vec<T, VEC>(qhi, after[0]);
        }
        if (full) {
#pragma unroll
            for (int t = 0; t < LB; ++t) load_vec<T, VEC>(src + (int64_t)t * m, x[t]);
        } else {
#pragma unroll
            for (int t = 0; t < LB; ++t) {
                if (r0 + t < rows) {
                    load_vec<T, VEC>(src + (int64_t)t * m, x[t]);
                } else {
#pragma unroll
                    for (int v = 0; v < VEC; ++v) x[t][v] = T(0);
                }
            }
        }
    };

    int g = b;
    if constexpr (GF)
        stage(lds, blob + sinv_at, a.sinv_bytes);
    else
        stage(lds, blob, blob_bytes);
    // flags bit 2: workgroups start out of step (b % 4 quarter steps of
    // `stagger` sleeps of 4096 cycles each), so that while some compute their
    // separators others stream, instead of every CU reaching its compute
    // phase at the same time
    if (a.flags & 4) {
        const int steps = (b % 4) * (a.flags >> 8);
        for (int i = 0; i < steps; ++i) __builtin_amdgcn_s_sleep(64);
    }
    __syncthreads();
    if (g < a.ngroups) load_group(g);
    const int q = lmap[p];  // stored copy of this block's factor, spikes and separator rows
    const Row *fr0 = lfac + q * LB;
    const T *sp0 = lspk + q * LB * 2 * H;
    const T *cf = lscf + q * H * NB;
    const T *cfp = lscf + lmap[pp] * H * NB;  // the previous block's separator rows
    // the separator rows' couplings to interior rows, the same for every
    // group: the own separator's to this block's last rows (c + d < H) and
    // the previous separator's to this block's first rows (c + d >= 2H)
    T cl[H][H], cr[H][H];
#pragma unroll
    for (int c = 0; c < H; ++c)
#pragma unroll
        for (int d = 0; d < H; ++d) {
            cl[c][d] = (c + d < H) ? cf[c * NB + d] : T(0);
            cr[c][d] = (2 * H - c + d < NB) ? cfp[c * NB + 2 * H - c + d] : T(0);
        }
    for (; g < a.ngroups; g += grid) {
        int step = 1;
        if constexpr (CN == 1 || CN == 2) step = a.steps;
        for (; step > 0; --step) {
            // the lane's offsets into the separator buffers, made opaque each
            // group so that the addresses derived from them are formed where they
            // are used instead of being kept live (and spilled) across the loop
            int o_own = s0 * ldr + H * p, o_prev = s0 * ldr + H * pp, o_col = s0 * ldr;
            asm volatile("" : "+v"(o_own), "+v"(o_prev), "+v"(o_col));
            // GF: the plan is read-only global memory, and its loads would be
            // hoisted out of the loop (every row's coefficients live at once)
            // unless its addresses are opaque here too
            const Row *fr = fr0;
            const T *sp = sp0;
            if constexpr (GF) asm volatile("" : "+v"(fr), "+v"(sp));

            if constexpr (SEG) {
                if (at_lo) {
#pragma unroll
                    for (int v = 0; v < VEC; ++v)
#pragma unroll
                        for (int t = 0; t < H; ++t)
#pragma unroll
                            for (int c = t; c < H; ++c) x[t][v] = fma(-clo[t][c], before[c][v], x[t][v]);
                }
                if (at_hi && full) {
#pragma unroll
                    for (int v = 0; v < VEC; ++v)
#pragma unroll
                        for (int t = 0; t < H; ++t)
#pragma unroll
                            for (int c = 0; c <= t; ++c)
                                x[NI + t][v] = fma(-chi[t][c], H == 1 ? after[c][v] : before[c][v], x[NI + t][v]);
                } else if (H == 1 && at_hi) {
                    // a ragged last segment of a periodic matrix
#pragma unroll
                    for (int t = 0; t < LB; ++t)
                        if (r0 + t == n - 1) {
#pragma unroll
                            for (int v = 0; v < VEC; ++v) x[t][v] = fma(-chi[0][0], after[0][v], x[t][v]);
                        }
                }
            }

            // 1. block sweeps (Section 3.1 / 4.1 recurrences, block factor);
            // each group of G rows reads its coefficients while the previous
            // group computes
            block_sweeps<KIND, T, LB, VEC, GF>(fr, x);
            // 2. the separator right-hand sides in two parts: the previous
            // separator takes minus its couplings to this block's first rows
            // (redr), the block's own separator takes f_sep minus its couplings to
            // this block's last interior rows (redl); one barrier.  (In this order
            // the first rows' values are dropped before the last rows' are used,
            // which keeps the FP64 pentadiagonal kernel within its registers.)
            if (has_prev) {
#pragma unroll
                for (int v = 0; v < VEC; ++v)
#pragma unroll
                    for (int c = 0; c < H; ++c) {
                        // band d = 2H - c + e of separator row c meets this block's row e
                        T yh = T(0);
#pragma unroll
                        for (int e = 0; e + 2 * H - c < NB; ++e) yh = fma(-cr[c][e], x[e][v], yh);
                        lredr[o_prev + v * ldr + c] = yh;
                    }
            }
            if (has_sep) {
#pragma unroll
                for (int v = 0; v < VEC; ++v)
#pragma unroll
                    for (int c = 0; c < H; ++c) {
                        // separator rows are identity rows of the block factor: the
                        // sweeps leave their right-hand sides in place
                        T yh = x[NI + c][v];
                        // band d < H - c of separator row c meets row NI + c + d - H
#pragma unroll
                        for (int d = 0; d + c < H; ++d) yh = fma(-cl[c][d], x[NI + c + d - H][v], yh);
                        lredl[o_own + v * ldr + c] = yh;
                    }
            }
            __syncthreads();
            // 3. separators
            T zr[H][VEC], zl[H][VEC];
            if (Nr == 0) {
#pragma unroll
                for (int c = 0; c < H; ++c)
#pragma unroll
                    for (int v = 0; v < VEC; ++v) zr[c][v] = zl[c][v] = T(0);
            } else if (MMA && blockDim.x % kWave == 0 &&
                       (!alias || ((Nr + 15) / 16) * ((S + 15) / 16) <= (int)(blockDim.x / kWave))) {
                if constexpr (MMA) {
                    // flags bit 6: every column of S^{-1}
                    const int kw = (a.flags & 64) ? 0 : a.kw;
                    if (alias)
                        sep_mma<true>(lsinv, lredl, lredr, lz, Nr, S, ldr, a.kofs, kw);
                    else
                        sep_mma<false>(lsinv, lredl, lredr, lz, Nr, S, ldr, a.kofs, kw);
                }
                __syncthreads();
#pragma unroll
                for (int c = 0; c < H; ++c)
#pragma unroll
                    for (int v = 0; v < VEC; ++v) {
                        // indices stay inside the separators even where unused
                        const T zo = lz[(has_sep ? o_own : o_col) + v * ldr + c];
                        const T zp = lz[(has_prev ? o_prev : o_col) + v * ldr + c];
                        zr[c][v] = has_sep ? zo : T(0);
                        zl[c][v] = has_prev ? zp : T(0);
                    }
                // the separators are redL's storage: the next group writes redL
                // only after every lane has read them
                if (alias) __syncthreads();
            } else {
                // rows of S^{-1} for the own and the previous separator (a block
                // without one reads the other's rows and discards the result)
                const T *rr = lsinv + (size_t)H * (a.periodic || p < P - 1 ? p : pp) * Nr;
                const T *rl = lsinv + (size_t)H * (a.periodic || p > 0 ? pp : p) * Nr;
                T ar[H][VEC], al[H][VEC];
#pragma unroll
                for (int c = 0; c < H; ++c)
#pragma unroll
                    for (int v = 0; v < VEC; ++v) ar[c][v] = al[c][v] = T(0);
                for (int k = 0; k < Nr; ++k) {
#pragma unroll
                    for (int v = 0; v < VEC; ++v) {
                        const T y = lredl[o_col + v * ldr + k] + lredr[o_col + v * ldr + k];
#pragma unroll
                        for (int c = 0; c < H; ++c) {
                            ar[c][v] = fma(rr[c * Nr + k], y, ar[c][v]);
                            al[c][v] = fma(rl[c * Nr + k], y, al[c][v]);
                        }
                    }
                }
#pragma unroll
                for (int c = 0; c < H; ++c)
#pragma unroll
                    for (int v = 0; v < VEC; ++v) {
                        zr[c][v] = has_sep ? ar[c][v] : T(0);
                        zl[c][v] = has_prev ? al[c][v] : T(0);
                    }
                // every lane has read redL / redR before the next group writes them
                __syncthreads();
            }
            // 4. correction and stores
            T *dst = out + (int64_t)r0 * m + col(g);
            const bool one = last_only(g);
            // the spikes of GC rows per round trip; from global memory (GF) the
            // next rows' spikes are loaded before the current rows are stored,
            // since a load issued after a store waits for that store
            constexpr int GC = GF ? 2 : G, NS = GF ? 2 : 1;
            T spt[NS][GC][2 * H];
            auto spikes = [&](int gr, T(&dstk)[GC][2 * H]) {
                if constexpr (GF) asm volatile("" : "+v"(sp));
#pragma unroll
                for (int u = 0; u < GC; ++u)
#pragma unroll
                    for (int k = 0; k < 2 * H; ++k) dstk[u][k] = sp[(gr * GC + u) * 2 * H + k];
            };
            if constexpr (GF) spikes(0, spt[0]);
#pragma unroll
            for (int gr = 0; gr < LB / GC; ++gr) {
                T(&cur)[GC][2 * H] = spt[GF ? gr & 1 : 0];
                if constexpr (GF) {
                    if (gr + 1 < LB / GC) spikes(gr + 1, spt[(gr + 1) & 1]);
                } else {
                    spikes(gr, cur);
                }
#pragma unroll
                for (int u = 0; u < GC; ++u) {
                    const int t = gr * GC + u;
                    T v2[VEC];
#pragma unroll
                    for (int v = 0; v < VEC; ++v) {
                        T val = x[t][v];
#pragma unroll
                        for (int c = 0; c < H; ++c) {
                            val = fma(-cur[u][c], zr[c][v], val);
                            val = fma(-cur[u][H + c], zl[c][v], val);
                        }
                        if (t >= NI) val = has_sep ? zr[t >= NI ? t - NI : 0][v] : val;
                        v2[v] = val;
                    }
                    if constexpr (CN) {
                        // computed here, not sunk past the barrier below (which
                        // would keep every row's spikes live until then)
#pragma unroll
                        for (int v = 0; v < VEC; ++v) {
                            x[t][v] = v2[v];
                            asm volatile("" : "+v"(x[t][v]));
                        }
                    } else if (full || r0 + t < rows) {
                        if (ANYM && one)
                            __builtin_nontemporal_store(v2[VEC - 1], dst + (int64_t)t * m + VEC - 1);
                        else
                            store_vec_nt<T, VEC>(dst + (int64_t)t * m, v2);
                    }
                }
                pin(zr[0][0]);
            }
            if constexpr (CN) {
                // 5. Crank-Nicolson output rows from the block's solution
#pragma unroll
                for (int v = 0; v < VEC; ++v)
#pragma unroll
                    for (int c = 0; c < H; ++c)
                        if (active) ltop[((s0 + v) * P + p) * H + c] = x[c][v];
                __syncthreads();
                const bool has_next = a.periodic || p < P - 1;
                const int pn = p == P - 1 ? 0 : p + 1;
                T dn[H][VEC];
#pragma unroll
                for (int v = 0; v < VEC; ++v)
#pragma unroll
                    for (int c = 0; c < H; ++c) {
                        const T t0 = ltop[((s0 + v) * P + pn) * H + c];
                        dn[c][v] = has_next ? t0 : T(0);
                    }
                if constexpr (SEG) {
                    if (at_hi) {
#pragma unroll
                        for (int v = 0; v < VEC; ++v)
#pragma unroll
                            for (int c = 0; c < H; ++c) dn[c][v] = H == 1 ? after[c][v] : before[c][v];
                        // the row after a ragged last segment (periodic)
                        if (H == 1 && !full) {
#pragma unroll
                            for (int t = 0; t < LB; ++t)
                                if (r0 + t == n) {
#pragma unroll
                                    for (int v = 0; v < VEC; ++v) x[t][v] = after[0][v];
                                }
                        }
                    }
                }
                // rows above the block: the previous block's separators (0 above
                // the first block of a matrix that does not wrap round)
                T up[H][VEC];  // the H rows above row t, before their own update
                T *q = dst;    // CN 3: stepped row by row, as below
#pragma unroll
                for (int c = 0; c < H; ++c)
#pragma unroll
                    for (int v = 0; v < VEC; ++v) up[c][v] = SEG && at_lo ? before[c][v] : zl[c][v];
#pragma unroll
                for (int t = 0; t < LB; ++t) {
                    T cb[NB];
#pragma unroll
                    for (int e = 0; e < NB; ++e) cb[e] = CN == 1 ? lband[(r0 + t) * NB + e] : (T)a.coef.c[e];
                    T v2[VEC];
#pragma unroll
                    for (int v = 0; v < VEC; ++v) {
                        T ax = T(0);
#pragma unroll
                        for (int e = 0; e < NB; ++e) {
                            const int i = t - H + e;
                            const T u = e < H ? up[e][v] : (i >= LB ? dn[i - LB][v] : x[i][v]);
                            ax = e == 0 ? cb[0] * u : fma(cb[e], u, ax);
                        }
                        v2[v] = T(2) * x[t][v] - ax;
#pragma unroll
                        for (int c = 0; c < H; ++c) up[c][v] = c + 1 < H ? up[c + 1][v] : x[t][v];
                    }
                    if constexpr (CN == 3) {
                        if (full || r0 + t < rows) store_vec_nt<T, VEC>(q, v2);
                        q += m;
                        asm volatile("" : "+v"(q));
                    } else {
                        // rows past the matrix stay 0
#pragma unroll
                        for (int v = 0; v < VEC; ++v) x[t][v] = full || r0 + t < rows ? v2[v] : T(0);
                    }
                    if (t % G == G - 1) pin(v2[0]);
                }
            }
        }
        if constexpr (CN && CN != 3) {
            // one store pointer stepped row by row (opaque, so that the rows'
            // addresses are not all formed up front and kept live)
            T *q = out + (int64_t)r0 * m + col(g);
            const bool one = last_only(g);
#pragma unroll
            for (int t = 0; t < LB; ++t) {
                if (full || r0 + t < rows) {
                    if (ANYM && one)
                        __builtin_nontemporal_store(x[t][VEC - 1], q + VEC - 1);
                    else
                        store_vec_nt<T, VEC>(q, x[t]);
                }
                q += m;
                asm volatile("" : "+v"(q));
            }
            if constexpr (SEG) {
                // the cut after the segment: c' = 2 u - A u = 2 u - c
                if (at_hi) {
                    T *qc = out + (int64_t)n * m + col(g);
#pragma unroll
                    for (int c = 0; c < H; ++c) {
                        T w[VEC];
                        load_vec<T, VEC>(qc + (int64_t)c * m, w);
#pragma unroll
                        for (int v = 0; v < VEC; ++v) w[v] = T(2) * (H == 1 ? after[c][v] : before[c][v]) - w[v];
                        if (ANYM && one)
                            __builtin_nontemporal_store(w[VEC - 1], qc + (int64_t)c * m + VEC - 1);
                        else
                            store_vec_nt<T, VEC>(qc + (int64_t)c * m, w);
                    }
                }
            }
        }
        if (g + grid < a.ngroups) load_group(g + grid);
    }
}

// The unknowns of the cut rows (the cut form's first kernel): for every cut and
// system, H rows of A^{-1} near the cut times the right-hand sides there, into
// the cut's rows.  A workgroup takes one cut and 64 * VEC systems; its four
// waves take a quarter of the window's rows each and add up in LDS (fixed
// order), so that the loads of a system, all independent, are in flight over
// four waves.  Reads what it needs of the right-hand sides once more than the
// solve does: 2 * 37 rows in 258 for the s = 0.5 hyperdiffusion matrix.  With
// ucut they go there, [cut][H][m], and the right-hand sides stay as they are.  The
// sums are FP64 whatever T is; the window of a cut holds no other cut's rows.
constexpr int kCutWaves = 4;

template <int H, typename T, int VEC>
__global__ __launch_bounds__(64 * kCutWaves) void k_cut_rows(const CutWin *__restrict__ wins, int ncuts, T *x,
                                                             int64_t m, int n, T *ucut) {
    const int lane = threadIdx.x % kWave, part = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const cptr<CutWin> win = (cptr<CutWin>)(wins + blockIdx.x % ncuts);
    const int64_t j0 = ((int64_t)(blockIdx.x / ncuts) * kWave + lane) * VEC, j = min(j0, m - VEC);
    const int per = (win->len + kCutWaves - 1) / kCutWaves;
    const int i0 = part * per, i1 = min(i0 + per, win->len);
    const cptr<double> w = (cptr<double>)win->w;
    const T *src = x + j;
    const int first = win->first;
    auto row = [&](int i) { return (int64_t)(first + i < n ? first + i : first + i - n) * m; };
    double z[H][VEC];
#pragma unroll
    for (int c = 0; c < H; ++c)
#pragma unroll
        for (int v = 0; v < VEC; ++v) z[c][v] = 0.0;
    constexpr int U = 8;
    int i = i0;
    for (; i + U <= i1; i += U) {
        T f[U][VEC];
#pragma unroll
        for (int u = 0; u < U; ++u) load_vec<T, VEC>(src + row(i + u), f[u]);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int c = 0; c < H; ++c)
#pragma unroll
                for (int v = 0; v < VEC; ++v) z[c][v] = fma(w[(i + u) * H + c], (double)f[u][v], z[c][v]);
    }
    for (; i < i1; ++i) {
        T f[VEC];
        load_vec<T, VEC>(src + row(i), f);
#pragma unroll
        for (int c = 0; c < H; ++c)
#pragma unroll
            for (int v = 0; v < VEC; ++v) z[c][v] = fma(w[i * H + c], (double)f[v], z[c][v]);
    }
    // every wave has read its rows (the cut's own among them) before any is written
    __shared__ double sum[kCutWaves][H][VEC][kWave];
#pragma unroll
    for (int c = 0; c < H; ++c)
#pragma unroll
        for (int v = 0; v < VEC; ++v) sum[part][c][v][lane] = z[c][v];
    __syncthreads();
    if (part >= H) return;
    T r[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
        double t = sum[0][part][v][lane];
#pragma unroll
        for (int q = 1; q < kCutWaves; ++q) t += sum[q][part][v][lane];
        r[v] = (T)t;
    }
    T *dst = ucut ? ucut + ((int64_t)(blockIdx.x % ncuts) * H + part) * m + j : x + (int64_t)(win->row + part) * m + j;
    // past the last pair: the last system only (see k_sep)
    if (VEC == 1 || j0 > m - VEC)
        dst[VEC - 1] = r[VEC - 1];
    else
        *reinterpret_cast<typename Pair<T>::type *>(dst) = typename Pair<T>::type{r[0], r[VEC - 1]};
}

// ---------------------------------------------------------------------------
// Launch side.

// Threads a workgroup may have: the lane's LB * VEC values take
// LB * VEC * sizeof(T) / 4 registers, and a CU's register file holds 512 per
// lane of one wave per SIMD.
template <typename T, int LB, int VEC>
constexpr int sep_maxt() {
    return LB * VEC * (int)sizeof(T) / 4 <= 64 ? 1024 : 512;
}

template <int KIND, typename T, int LB, int VEC, bool GF, int CN = 0, bool SEG = false>
hipError_t sep_kernel(const void **fn) {
    auto kern = k_sep<KIND, T, LB, VEC, sep_maxt<T, LB, VEC>(), GF, CN, SEG>;
    // once per instantiation; thread-safe static initialisation, so that
    // concurrent first launches from several host threads do not race
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                                       (int)kMaxPartLdsBytes);
    if (attr != hipSuccess) return attr;
    *fn = reinterpret_cast<const void *>(kern);
    return hipSuccess;
}

// The shapes built: (LB, VEC) with at most 128 registers of values per lane;
// with the plan in global memory (GF) the two longest, (32, 2) and (64, 1);
// Crank-Nicolson steps (plan in LDS) (16, 1), (32, 1), (32, 2) and (64, 1).
template <int KIND, typename T, int CN>
hipError_t sep_kernel_cn(int lb, int vec, const void **fn, int *maxt) {
    if (lb == 16 && vec == 1) return *maxt = sep_maxt<T, 16, 1>(), sep_kernel<KIND, T, 16, 1, false, CN>(fn);
    if (lb == 32 && vec == 1) return *maxt = sep_maxt<T, 32, 1>(), sep_kernel<KIND, T, 32, 1, false, CN>(fn);
    if (lb == 32 && vec == 2) return *maxt = sep_maxt<T, 32, 2>(), sep_kernel<KIND, T, 32, 2, false, CN>(fn);
    if (lb == 64 && vec == 1) return *maxt = sep_maxt<T, 64, 1>(), sep_kernel<KIND, T, 64, 1, false, CN>(fn);
    return hipErrorInvalidValue;
}

template <int KIND, typename T>
hipError_t sep_kernel_of(int lb, int vec, bool gf, int cn, const void **fn, int *maxt) {
    if (cn && gf) return hipErrorInvalidValue;
    if (cn == 1) return sep_kernel_cn<KIND, T, 1>(lb, vec, fn, maxt);
    if (cn == 2) return sep_kernel_cn<KIND, T, 2>(lb, vec, fn, maxt);
    if constexpr (KIND == SBS_PENTA)
        if (cn == 3) return sep_kernel_cn<KIND, T, 3>(lb, vec, fn, maxt);
    if (cn) return hipErrorInvalidValue;
    if (gf) {
        if (lb == 32 && vec == 2) return *maxt = sep_maxt<T, 32, 2>(), sep_kernel<KIND, T, 32, 2, true>(fn);
        if (lb == 64 && vec == 1) return *maxt = sep_maxt<T, 64, 1>(), sep_kernel<KIND, T, 64, 1, true>(fn);
        return hipErrorInvalidValue;
    }
    if (lb == 16 && vec == 1) return *maxt = sep_maxt<T, 16, 1>(), sep_kernel<KIND, T, 16, 1, false>(fn);
    if (lb == 16 && vec == 2) return *maxt = sep_maxt<T, 16, 2>(), sep_kernel<KIND, T, 16, 2, false>(fn);
    if (lb == 32 && vec == 1) return *maxt = sep_maxt<T, 32, 1>(), sep_kernel<KIND, T, 32, 1, false>(fn);
    if (lb == 32 && vec == 2) return *maxt = sep_maxt<T, 32, 2>(), sep_kernel<KIND, T, 32, 2, false>(fn);
    if (lb == 64 && vec == 1) return *maxt = sep_maxt<T, 64, 1>(), sep_kernel<KIND, T, 64, 1, false>(fn);
    if constexpr (sizeof(T) == 4)
        if (lb == 64 && vec == 2) return *maxt = sep_maxt<T, 64, 2>(), sep_kernel<KIND, T, 64, 2, false>(fn);
    return hipErrorInvalidValue;
}

hipError_t sep_fn(int kind, int tc, int lb, int vec, bool gf, int cn, const void **fn, int *maxt) {
    const int k = kind == SBS_PENTA ? SBS_PENTA : SBS_TRI;  // periodic blocks are plain tridiagonal
    if (k == SBS_TRI)
        return tc == 0 ? sep_kernel_of<SBS_TRI, double>(lb, vec, gf, cn, fn, maxt)
                       : sep_kernel_of<SBS_TRI, float>(lb, vec, gf, cn, fn, maxt);
    return tc == 0 ? sep_kernel_of<SBS_PENTA, double>(lb, vec, gf, cn, fn, maxt)
                   : sep_kernel_of<SBS_PENTA, float>(lb, vec, gf, cn, fn, maxt);
}

// LDS of one workgroup: the plan (GF: S^{-1} only), the two parts of the
// separator right-hand sides and (FP64: the matrix-core product's output)
// the separators, unless `alias` puts them in redL's storage; Crank-Nicolson
// steps add the blocks' first rows after a third buffer, and the band rows
// (cn 1).  H: the half band width, for those.
size_t sep_lds(const SepPlan &sp, int tc, int S, bool gf, bool alias, int cn = 0, int H = 0) {
    const size_t elem = tc == 0 ? 8 : 4;
    const size_t red = tc == 0 ? sep_red_bytes<double>(S, sp.Nr) : sep_red_bytes<float>(S, sp.Nr);
    const size_t plan = gf ? (tc == 0 ? sp.sinv_bytes64 : sp.sinv_bytes32) : sp.blob_bytes(tc);
    if (cn)
        return plan + 3 * red + ((size_t)S * sp.P * H * elem + 15) / 16 * 16 +
               (cn == 1 ? (size_t)sp.P * sp.lb * (2 * H + 1) * elem : 0);
    return plan + red * (tc == 0 && !alias ? 3 : 2);
}

int cu_count(int device) { return device_cus(device); }

// Checks one shape and fills in its launch figures; false if it cannot run.
// The plan goes to LDS whole where it fits with the group's buffers, else
// (or with flags bit 4) only S^{-1} does (GF), and where even that leaves no
// room for a third FP64 buffer the separators overwrite redL (flags bit 5,
// which only this function sets).
//
// cn: Crank-Nicolson steps with band rows (1) or constant bands (2), or one
// step with constant bands (3, pentadiagonal only); plan in LDS only.
bool sep_fit(const sbs_lhs *h, int tc, int64_t m, const void *x, int q, int vec, int S, int flags, SepChoice *c,
             int cn = 0) {
    const SepPlan &sp = h->sep[q];
    const size_t elem = tc == 0 ? 8 : 4;
    if (!sp.ok || m < vec || S < vec || S % vec) return false;
    if (vec == 2 && !cn && (m % 2 || reinterpret_cast<uintptr_t>(x) % (2 * elem))) return false;
    flags &= ~32;
    bool gf = (flags & 16) != 0, alias = false;
    if (cn && gf) return false;
    if (!cn && !gf && sep_lds(sp, tc, S, false, false) > kMaxPartLdsBytes) gf = true;
    if (!cn && gf && sep_lds(sp, tc, S, true, false) > kMaxPartLdsBytes) alias = tc == 0;
    const size_t lds = sep_lds(sp, tc, S, gf, alias, cn, h->kind == SBS_PENTA ? 2 : 1);
    if (lds > kMaxPartLdsBytes) return false;
    const void *fn = nullptr;
    int maxt = 0;
    if (sep_fn(h->kind, tc, sp.lb, vec, gf, cn, &fn, &maxt) != hipSuccess) return false;
    // whole waves, so that the matrix cores can form the separators (FP64), where these are
    // at least one row of tiles (pentadiagonal n = 400, m = 42058, 24 separators:
    // 65 us, with per-lane dot products 71; n = 274, m = 99320, 16: 115 and 121;
    // n = 160, 8 of them: 27 and 26 us, tridiagonal n = 72, m = 400000, 4: 98 and
    // 94 us; FP32 pentadiagonal n = 1536, m = 100 13.4 us, of 48 lanes 12.6)
    const int lanes = (S / vec) * sp.P;
    const int threads = tc == 0 && sp.Nr >= 16 ? (lanes + kWave - 1) / kWave * kWave : lanes;
    if (threads > maxt) return false;
    // the separators in redL: one matrix-core tile per wave
    if (alias && (lanes % kWave || ((sp.Nr + 15) / 16) * ((S + 15) / 16) > threads / kWave)) return false;
    int wgs = 0;
    if ((wgs = occupancy(fn, threads, lds)) < 1) return false;
    c->plan = q;
    c->vec = vec;
    c->S = S;
    c->threads = threads;
    c->lds = lds;
    c->wgs = wgs;
    c->flags = flags | (gf ? 16 : 0) | (alias ? 32 : 0);
    c->gf = gf;
    c->cn = cn;
    return true;
}

}  // namespace

// Default launch options: groups in launch order.
constexpr int kSepDefaultFlags = 0;

bool choose_sep(const sbs_lhs *h, int tc, int64_t m, const void *x, SepChoice *out, int cn) {
    const size_t elem = tc == 0 ? 8 : 4;
    const int cus = cu_count(h->device);
    SepChoice best;
    int64_t best_key[5] = {-1, -1, -1, -1, -1};
    for (int q = 2; q >= 0; --q)
        for (int vec = 2; vec >= 1; --vec)
            for (int S = 64; S >= 1; S /= 2) {
                SepChoice c;
                // two pentadiagonal FP64 systems per lane of 16 rows spill 40
                // registers: 32-row blocks instead (n = 300, m = 60000: 60 against
                // 93 us; n = 84, m = 90000 26 and 31 us), but not in short systems
                // or small batches, whose chain of rows the shorter blocks halve
                // (n = 40, m = 42058: 12.8 against 11.7 us; n = 84, m = 17928 12.3 and
                // 11.3 us; n = 57, m = 42058 14.1 and 14.2, n = 130 23.7 and 28.7)
                if (tc == 0 && h->kind == SBS_PENTA && vec == 2 && h->sep[q].lb == 16 && h->n > 56 &&
                    h->n * m > (int64_t(1) << 21))
                    continue;
                if (vec == 2 && (m % 2 || reinterpret_cast<uintptr_t>(x) % (2 * elem))) continue;  // pairs aligned
                if (!sep_fit(h, tc, m, x, q, vec, S, kSepDefaultFlags, &c, cn)) continue;
                const int64_t groups = (m + S - 1) / S;
                const int64_t engaged = std::min<int64_t>(groups, (int64_t)cus * c.wgs);
                // CUs engaged, the plan held in LDS, rows read in whole
                // 256-byte runs, 16-byte accesses, then lanes at work (up to
                // 8 waves per CU)
                const int64_t run = std::min<int64_t>((int64_t)S * elem, 256);
                const int64_t acc = (int64_t)vec * elem;
                const int64_t lanes = std::min<int64_t>(engaged * (S / vec * h->sep[q].P), (int64_t)cus * 8 * kWave);
                const int64_t key[5] = {std::min<int64_t>(engaged, cus), c.gf ? 0 : 1, run, acc, lanes};
                if (std::lexicographical_compare(best_key, best_key + 5, key, key + 5)) {
                    std::copy(key, key + 5, best_key);
                    best = c;
                }
            }
    if (best.plan < 0) return false;
    *out = best;
    return true;
}

// Several Crank-Nicolson steps run from registers, so the arithmetic, LDS reads
// and barriers of a step decide, not the row runs.  FP64, up to 4M unknowns:
// the shortest blocks (the serial chain of a step is two passes over a block),
// 8 systems per workgroup, 16 where that makes fewer than four waves (8 steps,
// tridiagonal n = 512, m = 2000: 30 us, 32-row blocks 38 to 42 us, the pair
// form 50 us; pentadiagonal 36, 49 and 69 us).  More than that: 32-row blocks
// with two systems per lane, which read each coefficient once for both, in the
// shape with the most waves resident per CU, 16 systems per workgroup on a tie
// (two workgroups then hide each other's barriers; tridiagonal n = 1000,
// m = 60000: 428 us, 32 systems 581 us, 16-row blocks 603 us, the pair form
// 774 us; pentadiagonal 540, 666, - and 672 us; with band rows in LDS n = 512
// 401 us at 64 systems, 883 us at 16; n = 1400, m = 20000, pentadiagonal: 347
// us at 16 systems, 556 us at 8, 64-row blocks 426 us).  64-row blocks where
// the separators of shorter ones leave too little LDS (pentadiagonal n = 2000,
// m = 10000: 254 us, the cut form 703, one launch of the sweeps per step 2007
// us).  Four systems per workgroup, 32-byte row runs, only for batches of up to
// 4M unknowns or without a cut form (n = 2000 with band rows, m = 10000: 851
// us, the cut form 660; m = 1000: 100 and 200 us).  Short systems have few lanes in
// a workgroup of 16 systems, so they take more, also of the shortest blocks
// (3 steps, pentadiagonal: n = 17, m = 500000 128 systems 54 us, 16 774 us, three
// launches of one step 117 us; n = 56, m = 300000 64 systems 93 us, 16 253 us;
// n = 200, m = 100001 64 systems 108 us, 16 141 us; tridiagonal n = 24, m = 100000
// 16-row blocks, 64 systems 19 us, 16 27 us; n = 32, m = 20000 32 systems 10.9 us,
// 16 12.0; n = 80 16.4 and 17.4 us).  FP32: one system per lane,
// 32-row blocks up to 8M unknowns, else 64-row ones in the widest workgroup of
// up to 12 waves (n = 1400, m = 40000: 32 systems 392 us, 16 517 us, 32-row
// blocks 746 us; n = 2000, m = 16000, 8 steps: 16 systems 192 us;
// a system of up to 32 rows is one 32-row block: pentadiagonal n = 22,
// m = 821696, 2 steps 47 us, as a 64-row one 84 us).
bool choose_sep_steps(const sbs_lhs *h, int tc, int64_t m, const void *x, int cn, SepChoice *out) {
    const int64_t unknowns = h->n * m;
    auto waves = [](const SepChoice &c) { return c.wgs * ((c.threads + kWave - 1) / kWave); };
    auto try_shape = [&](int q, int vec, int S, SepChoice *c) { return sep_fit(h, tc, m, x, q, vec, S, 0, c, cn); };
    // the shape of block length q with the most waves per CU, earlier S on a tie
    auto most = [&](int q, int vec, std::initializer_list<int> Ss, SepChoice *best) {
        bool any = false;
        for (int S : Ss) {
            SepChoice c;
            if (!try_shape(q, vec, S, &c) || (any && std::min(waves(c), 8) <= std::min(waves(*best), 8))) continue;
            *best = c;
            any = true;
        }
        return any;
    };
    SepChoice c;
    const bool cut = h->cut.P > 0;
    if (tc == 1) {
        if (unknowns > (int64_t(1) << 23)) {
            for (int S : {64, 32, 16})
                if (try_shape(h->n <= 32 ? 1 : 2, 1, S, &c) && c.threads <= 768) return *out = c, true;
        }
        return (most(1, 1, {h->n >= 512 ? 16 : 32, 16, 8}, &c) || most(2, 1, {16, 8}, &c) ||
                (!cut && most(2, 1, {4}, &c))) &&
               (*out = c, true);
    }
    const bool few = unknowns <= (int64_t(1) << 22);
    if (few) {
        const int P = h->sep[0].P, S = P >= 32 ? 8 : P <= 3 && m >= 65536 ? 64 : P <= 5 && m >= 8192 ? 32 : 16;
        if (try_shape(0, 1, S, &c) || try_shape(0, 1, 8, &c)) return *out = c, true;
    }
    if (!few && h->sep[1].P <= 7 && try_shape(1, 2, h->sep[1].P == 1 ? 128 : 64, &c)) return *out = c, true;
    if (!few && !h->sep[1].ok && h->sep[0].P <= 7 && try_shape(0, 1, 64, &c)) return *out = c, true;
    return ((m >= 2 && most(1, 2, {16, 32, 64}, &c)) || most(2, 1, {8, 16}, &c) || (m >= 2 && try_shape(1, 2, 8, &c)) ||
            ((few || !cut) && (most(2, 1, {4}, &c) || (m >= 2 && try_shape(1, 2, 4, &c)))) || try_shape(0, 1, 8, &c) ||
            try_shape(1, 1, 8, &c)) &&
           (*out = c, true);
}

bool sep_fills(const sbs_lhs *h, int tc, int64_t m, const SepChoice &c) {
    const size_t elem = tc == 0 ? 8 : 4;
    const int64_t groups = (m + c.S - 1) / c.S;
    return (size_t)c.S * elem >= 256 && groups >= cu_count(h->device);
}

bool sep_shape(const sbs_lhs *h, int tc, int64_t m, const void *x, int lb, int vec, int S, int flags, SepChoice *out) {
    for (int q = 0; q < 3; ++q)
        if (kPartLbs[q] == lb) return sep_fit(h, tc, m, x, q, vec, S, flags, out);
    return false;
}

namespace {

// The cut form's kernel: 32-row blocks, two systems per lane.
constexpr int kCutVec = 2;

template <int KIND, typename T>
hipError_t cut_kernel(int cn, const void **fn, int *maxt) {
    *maxt = sep_maxt<T, kSegLb, kCutVec>();
    return cn == 0   ? sep_kernel<KIND, T, kSegLb, kCutVec, false, 0, true>(fn)
           : cn == 1 ? sep_kernel<KIND, T, kSegLb, kCutVec, false, 1, true>(fn)
                     : sep_kernel<KIND, T, kSegLb, kCutVec, false, 2, true>(fn);
}

hipError_t cut_fn(int kind, int tc, int cn, const void **fn, int *maxt) {
    if (kind != SBS_PENTA)
        return tc == 0 ? cut_kernel<SBS_TRI, double>(cn, fn, maxt) : cut_kernel<SBS_TRI, float>(cn, fn, maxt);
    return tc == 0 ? cut_kernel<SBS_PENTA, double>(cn, fn, maxt) : cut_kernel<SBS_PENTA, float>(cn, fn, maxt);
}

template <int H, typename T>
hipError_t go_cut_rows(const CutPlan &cp, T *x, int64_t m, int64_t n, T *ucut, hipStream_t s) {
    const int64_t groups = (m + kWave * kCutVec - 1) / (kWave * kCutVec);
    if (groups * cp.cuts > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_cut_rows<H, T, kCutVec>), dim3((unsigned)(groups * cp.cuts)), dim3(kWave * kCutWaves), 0, s,
                       cp.wins, cp.cuts, x, m, (int)n, ucut);
    return hipGetLastError();
}

template <typename T>
hipError_t cut_rows(const sbs_lhs *h, void *x, int64_t m, void *ucut, hipStream_t s) {
    T *xt = static_cast<T *>(x), *ut = static_cast<T *>(ucut);
    return h->kind != SBS_PENTA ? go_cut_rows<1, T>(h->cut, xt, m, h->n, ut, s)
                                : go_cut_rows<2, T>(h->cut, xt, m, h->n, ut, s);
}

bool fit_cut(const sbs_lhs *h, int tc, int64_t m, int cn, CutChoice *out);

}  // namespace

// 128 systems per workgroup, one block per wave, so that every access of a wave
// is one run (1 KiB in FP64), if every CU then has a workgroup; else fewer
// (down to 64 bytes a run) until it has, or the workgroup is no longer whole
// waves.  Long runs are worth more than less reading by the windows or a
// second workgroup per CU: penta n = 1024, m = 65536 with segments of 256 rows
// and 128 systems 232 us, 256 rows and 64 systems (two workgroups) 255 us, 512
// rows and 64 systems 235 us, 32 systems 257 us; tri n = 1024 226, 249, 235
// and 257 us; FP32 tri n = 2000, m = 50001 218, 234, 311 us.
bool choose_cut(const sbs_lhs *h, int tc, int64_t m, CutChoice *out) { return fit_cut(h, tc, m, 0, out); }

bool choose_cut_cn(const sbs_lhs *h, int tc, int64_t m, int cn, CutChoice *out) { return fit_cut(h, tc, m, cn, out); }

namespace {

bool fit_cut(const sbs_lhs *h, int tc, int64_t m, int cn, CutChoice *out) {
    const CutPlan &cp = h->cut;
    const int H = h->kind == SBS_PENTA ? 2 : 1;
    if (cp.Q < 2 || m < kCutVec) return false;
    const size_t elem = tc == 0 ? 8 : 4;
    const void *fn = nullptr;
    int maxt = 0;
    if (cut_fn(h->kind, tc, cn, &fn, &maxt) != hipSuccess) return false;
    const int cus = cu_count(h->device);
    CutChoice best;
    for (int S = kWave * kCutVec; S * (int)elem >= 64; S /= 2) {
        CutChoice c;
        c.S = S;
        c.threads = S / kCutVec * cp.P;
        const size_t red = tc == 0 ? sep_red_bytes<double>(S, cp.Nr) : sep_red_bytes<float>(S, cp.Nr);
        c.lds = cp.blob_bytes[tc] + red * (tc == 0 || cn ? 3 : 2);
        if (cn)
            c.lds += ((size_t)S * cp.P * H * elem + 15) / 16 * 16 +
                     (cn == 1 ? (size_t)cp.P * kSegLb * (2 * H + 1) * elem : 0);
        if (c.threads > maxt || c.lds > kMaxPartLdsBytes) continue;
        if (best.S && c.threads % kWave) break;
        if ((c.wgs = occupancy(fn, c.threads, c.lds)) < 1) continue;
        best = c;
        if ((m + S - 1) / S * cp.Q >= cus) break;
    }
    if (!best.S) return false;
    *out = best;
    return true;
}

// One solve or Crank-Nicolson step (cn, with ucut): the cut rows, then the segments.
hipError_t run_cut(const sbs_lhs *h, const CutChoice &c, int tc, void *x, int64_t m, int cn, void *ucut,
                   hipStream_t s) {
    if (m <= 0) return hipSuccess;
    const CutPlan &cp = h->cut;
    const void *fn = nullptr;
    int maxt = 0;
    if (hipError_t e = cut_fn(h->kind, tc, cn, &fn, &maxt); e != hipSuccess) return e;
    const int64_t ngroups = (m + c.S - 1) / c.S;
    if (c.threads > maxt || ngroups * cp.Q > 0x7fffffff) return hipErrorInvalidValue;
    const hipError_t e = tc == 0 ? cut_rows<double>(h, x, m, ucut, s) : cut_rows<float>(h, x, m, ucut, s);
    if (e != hipSuccess) return e;
    SepMoreArgs a{};
    a.coef = h->coef;
    a.bands = h->bands;
    a.ucut = ucut;
    a.S = c.S;
    a.ngroups = (int)ngroups;
    a.steps = 1;
    a.m = m;
    a.segs = cp.segs;
    a.Q = cp.Q;
    // the GPU's workgroups shared out by the segments' rows (all but the last have
    // the same number) and what a group costs however few rows it has, about 48
    // rows (pentadiagonal n = 3124, m = 3736, a last segment of 28 rows: by the rows
    // alone four workgroups took its 30 groups in eight rounds, 69 us, now 53;
    // tridiagonal n = 2336, m = 12000 152 and 109 us; with 24 rows the first stays,
    // with 80 longer last segments take too many, n = 4660, m = 12000 199 and 206)
    constexpr int64_t kGroupRows = 48;
    const int64_t all = (int64_t)cu_count(h->device) * c.wgs, rows = cp.rows + kGroupRows;
    a.per = (int)std::max<int64_t>(1, std::min<int64_t>(ngroups, all * rows / (rows * (cp.Q - 1) + cp.last + kGroupRows)));
    a.per_last = (int)std::max<int64_t>(1, std::min<int64_t>(ngroups, all - (int64_t)a.per * (cp.Q - 1)));
    const unsigned char *blob = nullptr;
    void *args[] = {&blob, &a, &x, &x};
    return hipLaunchKernel(fn, dim3((unsigned)((int64_t)a.per * (cp.Q - 1) + a.per_last)), dim3(c.threads), args, c.lds, s);
}

}  // namespace

hipError_t launch_cut(const sbs_lhs *h, const CutChoice &c, int tc, void *x, int64_t m, hipStream_t s) {
    return run_cut(h, c, tc, x, m, 0, nullptr, s);
}

size_t cut_cn_bytes(const sbs_lhs *h, int tc, int64_t m) {
    return (size_t)h->cut.cuts * (h->kind == SBS_PENTA ? 2 : 1) * (size_t)m * (tc == 0 ? 8 : 4);
}

hipError_t launch_cut_cn(const sbs_lhs *h, const CutChoice &c, int tc, void *x, int64_t m, int cn, int steps, void *work,
                         hipStream_t s) {
    hipError_t e = hipSuccess;
    for (int k = 0; k < steps && e == hipSuccess; ++k) e = run_cut(h, c, tc, x, m, cn, work, s);
    return e;
}

hipError_t launch_sep(const sbs_lhs *h, const SepChoice &c, int tc, void *x, int64_t m, hipStream_t s, int steps) {
    if (m <= 0) return hipSuccess;
    const SepPlan &sp = h->sep[c.plan];
    const void *fn = nullptr;
    int maxt = 0;
    if (hipError_t e = sep_fn(h->kind, tc, sp.lb, c.vec, c.gf, c.cn, &fn, &maxt); e != hipSuccess) return e;
    if (c.threads > maxt) return hipErrorInvalidValue;
    const int64_t ngroups = (m + c.S - 1) / c.S;
    if (ngroups > 0x7fffffff) return hipErrorInvalidValue;
    SepMoreArgs a{};
    const bool f64 = tc == 0;
    a.fac_bytes = (int)(f64 ? sp.fac_bytes64 : sp.fac_bytes32);
    a.spk_bytes = (int)(f64 ? sp.spk_bytes64 : sp.spk_bytes32);
    a.scf_bytes = (int)(f64 ? sp.scf_bytes64 : sp.scf_bytes32);
    a.sinv_bytes = (int)(f64 ? sp.sinv_bytes64 : sp.sinv_bytes32);
    a.map_bytes = (int)sp.map_bytes;
    a.n = (int)h->n;
    a.P = sp.P;
    a.Nr = sp.Nr;
    a.S = c.S;
    a.ngroups = (int)ngroups;
    a.periodic = sp.periodic ? 1 : 0;
    a.flags = c.flags;
    a.kofs = sp.kofs;
    a.kw = sp.kw;
    a.steps = steps;
    a.m = m;
    a.coef = h->coef;
    a.bands = h->bands;
    const int grid = (int)std::min<int64_t>(ngroups, (int64_t)cu_count(h->device) * std::max(1, c.wgs));
    const unsigned char *blob = static_cast<const unsigned char *>(f64 ? sp.blob64 : sp.blob32);
    void *args[] = {&blob, &a, &x, &x};
    return hipLaunchKernel(fn, dim3(grid), dim3(c.threads), args, c.lds, s);
}

}  // namespace sbs
