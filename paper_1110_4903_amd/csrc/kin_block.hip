// kin_block.hip -- FP64 advance of mechanisms of 64 to 126 species with one cell on a workgroup of eight
// wavefronts, the cell's Newton matrix in their registers.
//
// A Newton iteration of such a cell is a chain of phases with a few thousand independent operations each,
// and a launch lasts as long as the chains of its cells.  Eight wavefronts shorten every phase, and a
// matrix in registers (101 x 102 entries: 52 of a lane's registers) leaves LDS for two cells on a compute
// unit, whose chains overlap; in LDS it would be 82 KB and one cell.  The phases:
//   * species functions, one species per thread, and the third-body concentrations, a slot's sum split
//     over several threads;
//   * reactions, one per thread: every reaction writes its terms dq/dc_k / M_k, q and dq/dT to LDS,
//     nothing is added there;
//   * the Jacobian in strips of 32 columns through LDS: the dense third-body terms, lanes along the columns
//     of a row; the other terms by gathering, each lane of a wavefront owning an entry and adding the
//     values that the host listed for it (LDS atomics would serialise on the popular species and sum in
//     no fixed order); then every wavefront takes its columns into registers, a row per lane and register
//     slot, and sums their part of the energy row;
//   * Gauss-Jordan elimination with partial pivoting: column k lies in wavefront k mod 8, which finds its
//     pivot, and publishes pivot and multipliers through LDS; all wavefronts take them to their columns
//     right of k.  Rows are never exchanged, a pivoted row is masked out of the search.  The lanes of rows
//     already pivoted would idle in a triangular elimination, so removing their entries too costs nothing
//     and leaves no back substitution.  The owner of column k + 1 brings it up to date first and
//     publishes, then takes part in the rest of step k: one barrier per step.
// Bound by the latency of a cell's chain of small steps, not by operations or bytes.  An iteration of a
// mechanism of 100 species and 600 reactions takes 220 k cycles of a block alone on a compute unit and 270 k for
// two blocks: elimination 140 k (1390 cycles a pivot: LDS 200, the first column 100, search and reciprocal 600,
// the other columns 400, of which a v_readlane_b32 takes ten cycles), third-body terms 37 k (4.5 rows use
// each row of efficiencies, from the vector cache at 21 bytes a cycle), gathering 18 k, rates 20 k.  2048 cells
// at 1 us: 57 ms in index order, 47 ms in cost order; on one wavefront per cell with the matrix in global
// memory 127 ms.
// Measured and not taken: panels of four columns per barrier (5500 cycles a panel: the wavefront that has
// factored one has its other columns still to do), pivot rows through LDS instead of v_readlane_b32 (LDS
// bound), four wavefronts, a block of 256 registers a lane alone on its compute unit.  Of 128 registers a lane
// the compiler spills 31 more (104 bytes of scratch; 21 and 64 below 95 species).
//
// Method as in the other layouts: Newton iterations on backward Euler in x = (Y, T) for a
// constant-(rho, e) cell, (I - hJ) dx = -G, dyadic sub-step halving on failure (Sec. 3.2, Eq.
// "kinetics"; Sec. 4.2, one independent system per cell).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "kin_internal.h"

namespace kin {
namespace {

#include "kin_xlane.h"

constexpr int kBW = kBlockWaves, kBT = 64 * kBW;   // wavefronts and threads of a block
constexpr int RW = 2;                              // rows of a lane: lane and lane + 64
constexpr int kStripLocal = kBlockStrip / kBW;     // columns of a strip that a wavefront takes
constexpr int kAhead = kBlockAhead;                // records or fours of efficiencies read at a time
constexpr int kSS = kBlockStrip + 1;               // odd row stride of a strip: a column is read bank by bank
// A wavefront has every kBW-th column: column `local` of its columns.
__device__ __forceinline__ int b_col(int wid, int local) { return local * kBW + wid; }

// Places of a block's arrays in its LDS, in doubles (the last ones hold ints), and the size of it all.
struct BPlaces {
    int V, S, c, g, hh, E, CV, M, X, XK, Mc, D, gt, lb, rp, dx, sc, xof, tq, ctl, size;
};

__host__ __device__ inline int b_even(int x) { return (x + 1) & ~1; }
// parts that a third-body concentration is summed in
__host__ __device__ inline int b_parts(int ntb) { return ntb > 0 ? (kBT / ntb < 1 ? 1 : (kBT / ntb > 8 ? 8 : kBT / ntb)) : 1; }

__host__ __device__ inline BPlaces b_places(const BlockTables &b, int ns, int nr, int ntb)
{
    const int N = ns + 1;
    BPlaces L;
    int p = 0;
    const auto take = [&](int n) { const int r = p; p += b_even(n); return r; };
    L.V = take((b.slots + 2) * nr + 1);
    // what only the rates need lies in the strip's place
    L.S = p;
    L.c = take(ns); L.g = take(ns); L.hh = take(ns);
    L.Mc = take(b_parts(ntb) * ntb); L.D = take(ntb);
    // and so do the multipliers
    L.lb = L.S;
    p = L.S + b_even(ns * kSS > p - L.S ? ns * kSS : p - L.S);   // (more than these need)
    L.E = take(ns); L.CV = take(ns); L.M = take(ns);
    L.X = take(N); L.XK = take(N);
    L.gt = take(8 * b.nquad); L.tq = take(4 * b.nquad);
    L.rp = take(64 * RW); L.dx = take(64 * RW);
    L.sc = take(48);
    L.xof = take(32 * RW); L.ctl = take(8);
    L.size = p;
    return L;
}

// The arrays themselves, as LDS pointers (a generic pointer would make every access a flat one).
typedef __attribute__((address_space(3))) double lds_d;
typedef __attribute__((address_space(3))) int lds_i;
typedef int b_int4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) b_int4 lds_4;
typedef __attribute__((address_space(3))) const char lds_c;
struct BLds {
    lds_d *V, *S, *c, *g, *hh, *E, *CV, *M, *X, *XK, *Mc, *D, *gt, *lb, *rp, *dx, *sc;
    lds_i *xof, *ctl, *tq;

    __device__ __forceinline__ BLds(const BPlaces &o, lds_d *p)
        : V(p + o.V), S(p + o.S), c(p + o.c), g(p + o.g), hh(p + o.hh), E(p + o.E), CV(p + o.CV), M(p + o.M), X(p + o.X), XK(p + o.XK),
          Mc(p + o.Mc), D(p + o.D), gt(p + o.gt), lb(p + o.lb), rp(p + o.rp), dx(p + o.dx), sc(p + o.sc),
          xof((lds_i *)(p + o.xof)), ctl((lds_i *)(p + o.ctl)),
          tq((lds_i *)(p + o.tq))
    {
    }
};

struct BThermo { double cp, h, s, dcp; };

__device__ __forceinline__ BThermo b_thermo(const WaveTables &t, int s, double T, double iT, double lT)
{
    const double *a = t.nasa + 14 * s + (T < t.Tmid[s] ? 0 : 7);
    BThermo o;
    o.cp = fma(T, fma(T, fma(T, fma(T, a[4], a[3]), a[2]), a[1]), a[0]);
    o.h = fma(a[5], iT, fma(T, fma(T, fma(T, fma(T, a[4] * 0.2, a[3] * 0.25), a[2] * (1.0 / 3.0)), a[1] * 0.5), a[0]));
    o.s = fma(a[0], lT, fma(T, fma(T, fma(T, fma(T, a[4] * 0.25, a[3] * (1.0 / 3.0)), a[2] * 0.5), a[1]), a[6]));
    o.dcp = fma(T, fma(T, fma(T, 4.0 * a[4], 3.0 * a[3]), 2.0 * a[2]), a[1]);
    return o;
}

// c^|nu| and its derivative for nu in 0..3, branch-free
__device__ __forceinline__ void b_pow(double c, int nu, double &p, double &dp)
{
    const double h = (nu >= 2 ? c : 1.0) * (nu >= 3 ? c : 1.0);
    p = (nu >= 1 ? c : 1.0) * h;
    dp = (double)nu * h;
}

// 1/x from the hardware reciprocal refined by two Newton steps (within an ulp for normal x)
__device__ __forceinline__ double b_recip(double x)
{
    double y = __builtin_amdgcn_rcp(x);
    y = fma(y, fma(-x, y, 1.0), y);
    return fma(y, fma(-x, y, 1.0), y);
}

template <typename T>
__device__ __forceinline__ T b_pick(const T (&v)[RW], int m)
{
    T r = v[0];
#pragma unroll
    for (int q = 1; q < RW; ++q) r = (m == q) ? v[q] : r;
    return r;
}

// Wave-wide maximum by DPP alone: within rows of 16, then along the rows to the last lane.
__device__ __forceinline__ unsigned wave_max_last(unsigned v)
{
    v = kmax(v, dpp<kDppX1>(v));
    v = kmax(v, dpp<kDppX2>(v));
    v = kmax(v, dpp<kDppHalfMirror>(v));
    v = kmax(v, dpp<kDppMirror>(v));
    v = kmax(v, dpp<0x142>(v));   // row_bcast:15
    v = kmax(v, dpp<0x143>(v));   // row_bcast:31
    return rdlane(v, 63);
}

// ctl words
enum { kCtlState, kCtlBad, kCtlPivot /* two */ };
// sc: 0.. partial c_v, 16.. partial d c_v / dT, then
enum { kScDe = 40, kScCf, kScH };

// Phases up to the reactions' values, at XK.
__device__ __forceinline__ void b_rates(const WaveTables &t, const BlockTables &b, const BLds &L, int tid, double rho)
{
    const int ns = t.ns, lane = tid & 63, wid = tid >> 6;
    const double T = L.XK[ns];
    const double iT = 1.0 / T, lT = log(T);
    const double rc = 1e-3 * rho, lPaRT = t.lnPaR - lT;
    // species functions; partial sums of c_v and its derivative, one per wavefront (64 species leave the
    // second of them a sum of nothing)
    if (wid < RW) {
        double cvp = 0.0, dcvp = 0.0;
        if (tid < ns) {
            const BThermo th = b_thermo(t, tid, T, iT, lT);
            const double im = b.iM[tid], rm = 8.31446261815324e3 * im, y = L.XK[tid];
            L.c[tid] = y * (rc * im);
            L.g[tid] = th.h - th.s;
            L.hh[tid] = th.h;
            L.E[tid] = rm * T * (th.h - 1.0);
            const double cv = rm * (th.cp - 1.0);
            L.CV[tid] = cv;
            cvp = y * cv;
            dcvp = y * (rm * th.dcp);
        }
        cvp = wave_sum(cvp);
        dcvp = wave_sum(dcvp);
        if (lane == 0) {
            L.sc[wid] = cvp;
            L.sc[16 + wid] = dcvp;
        }
    }
    if (tid == 0) L.ctl[kCtlBad] = 0;
    __syncthreads();
    // third-body concentrations [M]_q = sum_s eff_qs c_s
    const int parts = b_parts(t.ntb);
    if (t.ntb > 0) {
        for (int i = tid; i < parts * t.ntb; i += kBT) {
            const int part = i / t.ntb, q = i - part * t.ntb;
            double acc = 0.0;
#pragma unroll 20
            for (int s = part; s < ns; s += parts) acc = fma(t.effT[(size_t)s * t.ntb + q], L.c[s], acc);
            L.Mc[part * t.ntb + q] = acc;
        }
        __syncthreads();
    }
    const double4 *rxd4 = reinterpret_cast<const double4 *>(t.rxd);
    lds_c *cb = (lds_c *)L.c, *gb = (lds_c *)L.g, *hb = (lds_c *)L.hh;
    for (int r = tid; r < t.nr; r += kBT) {
        const RxnRec x = t.rxc[r];
        const double4 rd = rxd4[r];
        const RxnCoef *kc = t.rxk + r;
        const double lkf = fma(-rd.z, iT, fma(rd.y, lT, rd.x));
        const double dlkf = fma(rd.z, iT, rd.y) * iT;
        double pw[6], dpw[6], sg = 0.0, sh = 0.0;
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            pw[q] = 1.0;
            dpw[q] = 0.0;
            if (q < 3 ? q < b.rmax : q - 3 < b.pmax) {
                const double c = *(const lds_d *)(cb + x.coff[q]);
                const double nu = (double)x.nu[q];
                sg = fma(nu, *(const lds_d *)(gb + x.coff[q]), sg);
                sh = fma(nu, *(const lds_d *)(hb + x.coff[q]), sh);
                b_pow(c, q < 3 ? -x.nu[q] : x.nu[q], pw[q], dpw[q]);
            }
        }
        const double kf = exp(lkf);
        const double lKc = rd.w * lPaRT - sg;
        const double kb = exp(lkf - lKc);
        const double dlKc = (sh - rd.w) * iT;
        const bool rev = x.rev != 0;
        const double pf = kf * (pw[0] * pw[1] * pw[2]), pb = rev ? kb * (pw[3] * pw[4] * pw[5]) : 0.0;
        double dq[6];
        dq[0] = kf * (dpw[0] * pw[1] * pw[2]);
        dq[1] = kf * (pw[0] * dpw[1] * pw[2]);
        dq[2] = kf * (pw[0] * pw[1] * dpw[2]);
        dq[3] = rev ? -kb * (dpw[3] * pw[4] * pw[5]) : 0.0;
        dq[4] = rev ? -kb * (pw[3] * dpw[4] * pw[5]) : 0.0;
        dq[5] = rev ? -kb * (pw[3] * pw[4] * dpw[5]) : 0.0;
        double Mc = 1.0;
        const double D = pf - pb;
        if (x.tb >= 0) {
            Mc = 0.0;
            for (int p = 0; p < parts; ++p) Mc += L.Mc[p * t.ntb + x.tb];
            L.D[x.tb] = D;
        }
        lds_d *v = L.V + r;
        const auto put = [&](double x) {
            *v = x;
            v += t.nr;
        };
#pragma unroll
        for (int q = 0; q < 6; ++q)
            if (q < 3 ? q < b.rmax : q - 3 < b.pmax) put(Mc * dq[q] * kc->colc[q]);   // dQ/dc_k / M_k (zero for an unused slot)
        put(Mc * D);
        put(Mc * (pf * dlkf - pb * (dlkf - dlKc)));
    }
    __syncthreads();
    // third-body entries' factors nu D_q
    for (int e = tid; e < 8 * b.nquad; e += kBT) {
        const double nu = b.qnu[e];
        L.gt[e] = nu != 0.0 ? nu * L.D[b.qslot[e]] : 0.0;
    }
    __syncthreads();
}

// The augmented Newton matrix [I - hJ | -G] for a sub-step of size h from X, into A: rows lane, lane + 64,
// columns wid, wid + 8, ...
template <int NC>
__device__ __forceinline__ void b_system(const WaveTables &t, const BlockTables &b, const BLds &L, int tid, int wid, double rho,
                                         double h, double (&A)[RW][NC])
{
    const int ns = t.ns, N = ns + 1, lane = tid & 63;
    const double irc = 1.0 / (1e-3 * rho);
    bool bad = false;
    lds_c *Vb = (lds_c *)L.V;
    // a record word's terms: byte offset, and the sign in the lowest bit
    const auto signed_value = [&](unsigned off, unsigned sign) {
        const double v = *(const lds_d *)(Vb + off);
        return __hiloint2double(__double2hiint(v) ^ (int)sign, __double2loint(v));
    };
    const auto lo = [&](unsigned w) { return signed_value(w & 0xfff8u, w << 31); };
    const auto hi = [&](unsigned w) { return signed_value((w >> 16) & 0xfff8u, (w << 15) & 0x80000000u); };
    const int tc = tid & (kBlockStrip - 1);
#pragma unroll 1
    for (int st = 0; st < NC / kStripLocal; ++st) {
        const int c0 = st * kBlockStrip;
        // the wavefront's first records of this strip, wanted behind the barrier
        const auto *first = uniform_table(b.gfirst) + st * kBW + wid;
        const int r0 = first[0], r1 = first[1];
        uint4 w[kAhead];
        const auto records = [&](int r) {
#pragma unroll
            for (int q = 0; q < kAhead; ++q) w[q] = b.rec[(unsigned)((r + q) * 64 + lane)];
        };
        records(r0);
        // dense third-body terms of column c0 + tc: half a wavefront per row, kAhead fours of efficiencies of
        // both halves at a time (the cache answers in some 700 cycles)
        {
            const bool in = c0 + tc < ns;
            const unsigned ec = 8u * (st * t.ntb * kBlockStrip + tc);
            const int half = (tid >> 5) & 1;
            double acc = 0.0;
            const int q1 = uniform_table(b.qfirst)[wid + 1];
            for (int q0 = uniform_table(b.qfirst)[wid]; q0 < q1; q0 += kAhead) {
                double f[kAhead][4];
                int flag[kAhead];
#pragma unroll
                for (int k = 0; k < kAhead; ++k) {
                    const b_int4 o = *(const lds_4 *)(L.tq + 4 * (2 * (q0 + k) + half));
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        f[k][q] = *reinterpret_cast<const double *>(reinterpret_cast<const char *>(b.effQ) + ((unsigned)o[q] + ec));
                    flag[k] = uniform_table(b.qrow)[q0 + k];
                }
#pragma unroll
                for (int k = 0; k < kAhead; ++k) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) acc = fma(L.gt[4 * (2 * (q0 + k) + half) + q], f[k][q], acc);
                    if (flag[k] & 0x10000) {
                        const int row = (half ? flag[k] >> 8 : flag[k]) & 0xff;
                        if (row != 0xff) L.S[row * kSS + tc] = in ? acc : 0.0;
                        acc = 0.0;
                    }
                }
            }
        }
        __syncthreads();
        {
            double acc = 0.0;
            unsigned d = 0;
            for (int r = r0; r < r1; r += kAhead) {
                if (r != r0) records(r);
#pragma unroll
                for (int q = 0; q < kAhead; ++q)
                    if (r + q < r1) {
                        const int n = uniform_table(b.gterms)[r + q];   // places | 0x100 first record of its group | 0x200 last
                        if (n & 0x100) {
                            acc = hi(w[q].x);
                            d = w[q].x & 0xffffu;
                        } else {
                            acc += lo(w[q].x);
                            acc += hi(w[q].x);
                        }
                        if ((n & 0xff) > 2) {
                            const double v2 = lo(w[q].y), v3 = hi(w[q].y);
                            acc += v2;
                            acc += v3;
                        }
                        if ((n & 0xff) > 4) {
                            const double v4 = lo(w[q].z), v5 = hi(w[q].z), v6 = lo(w[q].w), v7 = hi(w[q].w);
                            acc += v4; acc += v5; acc += v6; acc += v7;
                        }
                        if ((n & 0x200) && d != 0xffffu) L.S[d] += acc;
                    }
            }
        }
        __syncthreads();
        // the wavefront's columns of the strip, behind those that it has
#pragma unroll
        for (int kk = 0; kk + kStripLocal < NC; ++kk)
#pragma unroll
            for (int m = 0; m < RW; ++m) A[m][kk] = A[m][kk + kStripLocal];
#pragma unroll
        for (int i = 0; i < kStripLocal; ++i) {
            const int kk = NC - kStripLocal + i;
            const int tcol = b_col(wid, i), col = c0 + tcol;
            double e = 0.0, v[RW];
#pragma unroll
            for (int m = 0; m < RW; ++m) {
                const int s = lane + 64 * m;
                double a = 0.0;
                v[m] = 0.0;
                if (s < ns && col <= N) {
                    v[m] = L.S[s * kSS + tcol] * L.M[s];
                    if (col >= ns) v[m] *= irc;
                    a = col == N ? -((L.XK[s] - L.X[s]) - h * v[m]) : (s == col ? 1.0 : 0.0) - h * v[m];
                    bad = bad || !__builtin_isfinite(a);
                }
                e = fma(s < ns ? L.E[s] : 0.0, v[m], e);
                A[m][kk] = a;
            }
            e = wave_sum(e);
            if (col == N) {
                const double f = wave_sum(fma(64 + lane < ns ? L.CV[64 + lane] : 0.0, v[1], L.CV[lane] * v[0]));
                if (lane == 0) {
                    L.sc[kScDe] = e;
                    L.sc[kScCf] = f;
                }
            }
            if (lane == 0 && col <= N) L.dx[col] = e;
        }
        __syncthreads();
    }
    // the energy row, a column per thread (in the place of the second column's multipliers)
    lds_d *erow = L.lb + 64 * RW;
    if (tid <= N) {
        const double cv = L.sc[0] + L.sc[1], dcv = L.sc[16] + L.sc[17];
        const double icv = 1.0 / cv, fT = -L.sc[kScDe] * icv, acc = L.dx[tid];
        double a;
        if (tid == N) {
            a = -((L.XK[ns] - L.X[ns]) - h * fT);
        } else {
            const double v = tid < ns ? -fma(fT, L.CV[tid], acc) * icv : -fma(fT, dcv, acc + L.sc[kScCf]) * icv;
            a = (tid == ns ? 1.0 : 0.0) - h * v;
        }
        bad = bad || !__builtin_isfinite(a);
        erow[tid] = a;
    }
    __syncthreads();
    if (lane == ns - 64)
#pragma unroll
        for (int kk = 0; kk < NC; ++kk) {
            const int col = b_col(wid, kk);
            if (col <= N) A[1][kk] = erow[col];
        }
    if (__any(bad) && lane == 0) L.ctl[kCtlBad] = 1;
}

// Gauss-Jordan elimination of A; afterwards column N, the first of its wavefront, holds u_kk x_k in the row
// that was pivot k.
// The pivot of a column is the largest entry by the leading 32 bits of its magnitude (exponent and 20
// bits): a multiplier is then at most 1 + 2^-20, and the search is one 32-bit reduction.  The error of the
// solution, against LU with pivots by all bits (101 unknowns): Newton matrices of condition up to 1e19, median
// 1.8e-9 to 2.6e-8 and 1.5e-9 to 7.5e-8; graded random matrices 3.0e-12 and 2.5e-12.
template <int NC>
__device__ __forceinline__ void b_eliminate(const BLds &L, int N, int lane, int wid, double (&A)[RW][NC])
{
    unsigned open[RW];   // all ones but the sign where the lane's row has not been a pivot, else zero
#pragma unroll
    for (int m = 0; m < RW; ++m) open[m] = lane + 64 * m < N ? 0x7fffffffu : 0u;
    // pivot and multipliers of column k, the wavefront's first
    const auto publish = [&](int k) {
        unsigned key[RW];
#pragma unroll
        for (int m = 0; m < RW; ++m) key[m] = (unsigned)__double2hiint(A[m][0]) & open[m];
        const unsigned best = wave_max_last(kmax(key[0], key[1]));
        const unsigned long long b0 = __builtin_amdgcn_uicmp(key[0], best, 32), b1 = __builtin_amdgcn_uicmp(key[1], best, 32);
        const bool hi = b0 == 0;
        const int w = __builtin_ctzll(hi ? b1 : b0) & 63;
        const double rp = b_recip(rdlane(hi ? A[1][0] : A[0][0], w));
        lds_d *lb = L.lb + (k & 1) * (64 * RW);
        lb[lane] = lane == w && !hi ? 0.0 : A[0][0] * rp;
        lb[lane + 64] = lane == w && hi ? 0.0 : A[1][0] * rp;
        if (lane == 0) {
            const int row = w + (hi ? 64 : 0);
            L.ctl[kCtlPivot + (k & 1)] = row;
            L.rp[row] = rp;
            L.xof[row] = k;
            if (best == 0) L.ctl[kCtlBad] = 1;   // (row may have been a pivot before: what follows is not used)
        }
    };
    const auto step = [&](int k, int next, int left) {   // next: the wavefront of column k + 1, its first now
        const bool own = wid == next && k + 1 < N;
        if (own) __builtin_amdgcn_s_setprio(3);   // the others wait for it
        const lds_d *lb = L.lb + (k & 1) * (64 * RW);
        const double l0 = lb[lane], l1 = lb[lane + 64];
        const int pr = __builtin_amdgcn_readfirstlane(L.ctl[kCtlPivot + (k & 1)]), p = pr & 63;
        const bool hi = pr >= 64;
        open[0] = lane == p && !hi ? 0u : open[0];
        open[1] = lane == p && hi ? 0u : open[1];
        // columns c0 .. c0 + n - 1 (the branch holds the reads alone: the updates stay in place)
        const auto update = [&](auto c0, auto nc) {
            constexpr int C = decltype(c0)::value, n = decltype(nc)::value;
            double u[n];
            if (hi) {
#pragma unroll
                for (int q = 0; q < n; ++q) u[q] = rdlane(A[1][C + q], p);
            } else {
#pragma unroll
                for (int q = 0; q < n; ++q) u[q] = rdlane(A[0][C + q], p);
            }
#pragma unroll
            for (int q = 0; q < n; ++q) {
                A[0][C + q] = fma(-l0, u[q], A[0][C + q]);
                A[1][C + q] = fma(-l1, u[q], A[1][C + q]);
            }
        };
        update(std::integral_constant<int, 0>{}, std::integral_constant<int, 1>{});
        if (own) {
            publish(k + 1);
            __builtin_amdgcn_s_setprio(0);
        }
        update(std::integral_constant<int, 1>{}, std::integral_constant<int, 3>{});
        if (left > 4) update(std::integral_constant<int, 4>{}, std::integral_constant<int, 4>{});
        if (left > 8) update(std::integral_constant<int, 8>{}, std::integral_constant<int, 4>{});
        if constexpr (NC > 12)
            if (left > 12) update(std::integral_constant<int, 12>{}, std::integral_constant<int, 4>{});
        __syncthreads();
    };
    // The next column is brought up to date and published first.  Eight steps take the first column of each
    // wavefront, then the columns move up by one: one copy of the code serves all steps (unrolled over the
    // columns it would not fit in the instruction cache), and a wavefront whose first column has been taken
    // goes on updating what is left of it.
    if (wid == 0) publish(0);
    __syncthreads();
    int left = N / kBW + 1;   // columns that a wavefront may have
#pragma unroll 1
    for (int k0 = 0; k0 < N; k0 += kBW) {
#pragma unroll 1
        for (int k = k0; k < k0 + kBW - 1 && k < N; ++k) step(k, k - k0 + 1, left);
        if (k0 + kBW > N) break;
#pragma unroll
        for (int c = 0; c + 1 < NC; ++c)
#pragma unroll
            for (int m = 0; m < RW; ++m) A[m][c] = A[m][c + 1];
        step(k0 + kBW - 1, 0, --left);
    }
}

// Mixture e and c_v at T of the state xk[] (one wavefront; every lane returns the same)
__device__ __forceinline__ void b_energy(const WaveTables &t, const BlockTables &b, int lane, const double (&x)[RW], double T,
                                         double &e, double &cv)
{
    double es = 0.0, cs = 0.0;
    const double iT = 1.0 / T;
#pragma unroll
    for (int m = 0; m < RW; ++m) {
        const int s = lane + 64 * m;
        if (s < t.ns) {
            const BThermo th = b_thermo(t, s, T, iT, 0.0);
            const double rm = 8.31446261815324e3 * b.iM[s];
            es = fma(x[m], rm * T * (th.h - 1.0), es);
            cs = fma(x[m], rm * (th.cp - 1.0), cs);
        }
    }
    e = wave_sum(es);
    cv = wave_sum(cs);
}

__device__ __forceinline__ bool b_invert_T(const WaveTables &t, const BlockTables &b, int lane, const double (&x)[RW], double e0,
                                           double T0, double &T_out)
{
    double T = T0, e, cv;
    for (int it = 0; it < 20; ++it) {
        b_energy(t, b, lane, x, T, e, cv);
        if (!(cv > 0.0)) break;
        const double dT = (e - e0) / cv;
        T -= dT;
        if (!__builtin_isfinite(T) || T < kTmin || T > kTmax) break;
        if (fabs(dT) <= 1e-13 * T) { T_out = T; return true; }
    }
    double lo = kTmin, hi = kTmax;
    b_energy(t, b, lane, x, lo, e, cv);
    const double flo = e - e0;
    b_energy(t, b, lane, x, hi, e, cv);
    const double fhi = e - e0;
    if (!(flo <= 0.0 && fhi >= 0.0)) return false;
    for (int it = 0; it < 200 && hi - lo > 1e-13 * lo; ++it) {
        const double mid = 0.5 * (lo + hi);
        b_energy(t, b, lane, x, mid, e, cv);
        if (e - e0 > 0.0) hi = mid; else lo = mid;
    }
    T_out = 0.5 * (lo + hi);
    return true;
}

// Add a zero that the compiler does not know to each pointer
template <typename... P> __device__ __forceinline__ void afresh(size_t z, P &...p)
{
    (..., (p += z));
}

// One block per cell, from the launch's cell `first` on; the hardware dispatcher balances cells of very
// different iteration counts.  The wavefront with the right-hand side holds the cell's state and decides; ctl and sc tell the others whether
// to go on and the sub-step size.
template <int NC>
__global__ void __launch_bounds__(kBT, 4) block_kernel(WaveTables t, BlockTables b, AdvanceArgs a, long long first)
{
    extern __shared__ double bsmem[];
    const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ns = t.ns, N = ns + 1;
    const BLds L(b_places(b, ns, t.nr, t.ntb), (lds_d *)bsmem);
    const int cw = N % kBW;   // the wavefront of column N
    const long long gi = first + blockIdx.x;
    if (gi >= a.total) return;
    int j = 0;
    while (j + 1 < a.nspan && a.span[j + 1].start <= gi) ++j;
    const long long ld = a.span[j].n;
    long long cell = gi - a.span[j].start;
    if (a.span[j].order) {
        const long long c = a.span[j].order[cell];
        if ((unsigned long long)c < (unsigned long long)ld) cell = c;
    }
    const double dt = a.span[j].dt;
    const Arena ar = arena_at(a.span[j].base, ld, ns);
    const double rho = ar.rho[cell], e0 = ar.e0[cell], T0 = ar.T[cell];
    if (tid == 0) L.V[(b.slots + 2) * t.nr] = 0.0;   // what the lists' padding reads
    for (int i = tid; i < ns; i += kBT) L.M[i] = t.M[i];
    for (int i = tid; i < 8 * b.nquad; i += kBT) L.tq[i] = 8 * kBlockStrip * b.qslot[i];   // byte offset of the slot's row
    bool fin = true;
#pragma unroll
    for (int m = 0; m < RW; ++m) {
        const int i = lane + 64 * m;
        double x = 0.0;
        if (i < ns) x = ar.Y[(size_t)i * ld + cell];
        else if (i == ns) x = T0;
        fin = fin && __builtin_isfinite(x);
        if (wid == cw && i < N) L.X[i] = L.XK[i] = x;
    }
    ScheduleTrace tr;
    if (wid == cw) tr.start(a.trace, a.trace_words, a.span[j].start + cell);
    // every wavefront has read the whole state, so they agree
    if (__any(!fin) || !__builtin_isfinite(rho) || !(rho > 0.0) || !__builtin_isfinite(e0) || !__builtin_isfinite(dt) ||
        !(dt >= 0.0) || T0 < kTmin || T0 > kTmax) {
        if (tid == 0) {
            ar.status[cell] = 3;
            ar.level[cell] = 0;
            ar.iters[cell] = 0;
            ar.sched[cell] = 0xcbf29ce484222325ull;
        }
        if (wid == cw) tr.finish(lane);
        return;
    }
    const bool adapt = a.L_forced < 0;
    const int Lc = adapt ? a.L_max : a.L_forced;
    const unsigned long long end = 1ull << Lc;
    unsigned long long tt = 0, hsh = 0xcbf29ce484222325ull;
    int l = adapt ? 0 : a.L_forced, level = l, iters = 0, k = 0, st = -1;
    bool failed = false;
    double r_prev = -1.0;
    double h = ldexp(dt, -l);
    __syncthreads();
    for (;;) {
        // what the iterations share of address arithmetic and table loads is computed again in each of them:
        // hoisted out of the loop it would not fit in the registers beside the matrix
        int it = tid;
        asm volatile("" : "+v"(it));
        const int lane = it & 63;
        size_t z = 0;
        asm volatile("" : "+s"(z));
        WaveTables tz = t;
        BlockTables bz = b;
        afresh(z, tz.nasa, tz.Tmid, tz.M, tz.rxd, tz.rxc, tz.rxk, tz.effT, bz.gfirst, bz.gterms, bz.rec, bz.qfirst, bz.qrow, bz.iM, bz.effQ,
               bz.qslot, bz.qnu);
        b_rates(tz, bz, L, it, rho);
        double A[RW][NC];
        b_system<NC>(tz, bz, L, it, wid, rho, h, A);
        b_eliminate<NC>(L, N, lane, wid, A);
        if (wid == cw) {
            double dx[RW], xk[RW];
            // a column without a pivot leaves rows that were none either: their xof was never written
            const bool ok = L.ctl[kCtlBad] == 0;
            if (ok) {
#pragma unroll
                for (int m = 0; m < RW; ++m) {
                    const int i = lane + 64 * m;
                    if (i < N) L.dx[L.xof[i]] = A[m][0] * L.rp[i];
                }
            }
            wave_sync();
#pragma unroll
            for (int m = 0; m < RW; ++m) {
                const int i = lane + 64 * m;
                dx[m] = i < N ? L.dx[i] : 0.0;
                xk[m] = i < N ? L.XK[i] : 0.0;
            }
            ++iters;
            if (k == 0) r_prev = -1.0;
            int outcome = 0;   // 0 go on, 1 accepted, 2 the attempt failed
            if (!ok) {
                outcome = 2;
            } else {
                bool conv = true, finx = true;
                double r = 0.0;
#pragma unroll
                for (int m = 0; m < RW; ++m) {
                    const int i = lane + 64 * m;
                    if (i < N) {
                        xk[m] += dx[m];
                        finx = finx && __builtin_isfinite(xk[m]);
                        const double tol = (i < ns ? a.atol_Y : a.atol_T) + a.rtol * fabs(xk[m]);
                        conv = conv && fabs(dx[m]) <= tol;
                        r = fmax(r, fabs(dx[m]) / tol);
                    }
                }
                const double Tk = rdlane(b_pick(xk, ns >> 6), ns & 63);
                const bool allconv = __all(conv);
                if (__any(!finx) || Tk < kTmin || Tk > kTmax) {
                    outcome = 2;
                } else if (!allconv && !a.point_implicit) {
                    if (a.diverge_ratio > 0.0) {
                        const double rw = wave_max(r);
                        if (r_prev >= 0.0 && rw > a.diverge_ratio * r_prev) outcome = 2;
                        else r_prev = rw;
                    }
                } else {
                    bool neg = false;
#pragma unroll
                    for (int m = 0; m < RW; ++m)
                        if (lane + 64 * m < ns) neg = neg || xk[m] < -a.y_neg;
                    double Tn;
                    if (!a.point_implicit && __any(neg)) {
                        outcome = 2;
                    } else if (!b_invert_T(t, b, lane, xk, e0, Tk, Tn)) {
                        outcome = 2;
                    } else {
                        outcome = 1;
#pragma unroll
                        for (int m = 0; m < RW; ++m)
                            if (lane + 64 * m == ns) xk[m] = Tn;
                    }
                }
            }
            if (outcome == 0 && ++k >= a.k_max) outcome = 2;
            if (outcome != 0) {
                hsh = (hsh ^ (unsigned long long)(2 * l + (outcome == 1 ? 1 : 0))) * 0x100000001b3ull;
                tr.add(outcome == 1, lane);
                k = 0;
                if (outcome == 1) {
#pragma unroll
                    for (int m = 0; m < RW; ++m)
                        if (lane + 64 * m < N) L.X[lane + 64 * m] = xk[m];
                    tt += 1ull << (Lc - l);
                    if (adapt && l > 0 && (tt & ((1ull << (Lc - l + 1)) - 1ull)) == 0ull) --l;
                    if (tt >= end) st = failed ? 1 : 0;
                } else {
#pragma unroll
                    for (int m = 0; m < RW; ++m)
                        if (lane + 64 * m < N) xk[m] = L.X[lane + 64 * m];
                    if (!adapt) {
                        st = 2;
                    } else {
                        failed = true;
                        ++l;
                        if (l > level) level = l;
                        if (l > a.L_max) { level = a.L_max; st = 2; }
                    }
                }
                if (st < 0 && iters >= a.max_iters) st = 2;
            }
#pragma unroll
            for (int m = 0; m < RW; ++m)
                if (lane + 64 * m < N) L.XK[lane + 64 * m] = xk[m];
            if (lane == 0) {
                L.ctl[kCtlState] = st;
                L.sc[kScH] = ldexp(dt, -l);
            }
        }
        __syncthreads();
        if (L.ctl[kCtlState] >= 0) break;
        h = L.sc[kScH];
    }
    if (wid != cw) return;
    if (st < 2) {
#pragma unroll
        for (int m = 0; m < RW; ++m) {
            const int i = lane + 64 * m;
            if (i < ns) ar.Y[(size_t)i * ld + cell] = L.X[i];
            else if (i == ns) ar.T[cell] = L.X[i];
        }
    }
    if (lane == 0) {
        ar.status[cell] = st;
        ar.level[cell] = level;
        ar.iters[cell] = iters;
        ar.sched[cell] = hsh;
    }
    tr.finish(lane);
}

}  // namespace

size_t block_lds_bytes(const WaveTables &t, const BlockTables &b)
{
    return sizeof(double) * (size_t)b_places(b, t.ns, t.nr, t.ntb).size;
}

// NC: columns of a wavefront, a multiple of those of a strip
template <int NC>
static hipError_t launch_nc(size_t lds, const WaveTables &t, const BlockTables &b, const AdvanceArgs &a, hipStream_t s)
{
    // above the 64 KiB that a kernel may take by default
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&block_kernel<NC>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    // a grid holds less than 2^32 threads, so the cells go in parts of half as many
    constexpr long long kPart = (1ll << 31) / kBT;
    for (long long first = 0; first < a.total; first += kPart) {
        const long long n = a.total - first < kPart ? a.total - first : kPart;
        hipLaunchKernelGGL((block_kernel<NC>), dim3((unsigned)n), dim3(kBT), lds, s, t, b, a, first);
        const hipError_t le = hipGetLastError();
        if (le != hipSuccess) return le;
    }
    return hipSuccess;
}

hipError_t launch_block(const WaveTables &t, const BlockTables &b, const AdvanceArgs &a, hipStream_t s)
{
    if (a.total <= 0) return hipSuccess;
    if (t.ns < kBlockNsMin || t.ns > kBlockNsMax) return hipErrorInvalidValue;
    const size_t lds = block_lds_bytes(t, b);
    switch ((t.ns + 2 + kBlockStrip - 1) / kBlockStrip) {
    case 3: return launch_nc<3 * kStripLocal>(lds, t, b, a, s);
    case 4: return launch_nc<4 * kStripLocal>(lds, t, b, a, s);
    }
    return hipErrorInvalidConfiguration;
}

}  // namespace kin
