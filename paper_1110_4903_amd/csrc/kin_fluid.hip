// kin_fluid.hip -- the fluid step of the operator-split reactive Euler solver (Sec. 3.1), on a
// 2-D grid whose cells hold the conserved variables of Sec. 2, Q = (rho_s [Ns], rho u, rho v, E),
// E = sum_s rho_s e_s + rho |u|^2 / 2 with each species' energy taken without its formation
// energy, e_s(T) = e_s^NASA(T) - e_s^NASA(T_ref), T_ref = 298.15 K (Sec. 2, Eq. energy); the
// chemistry sub-step of the split (the conserved-variable adapter) uses the same energy.
//
// A step is dimensionally split: an x sweep then a y sweep (or the reverse).  A sweep is three
// Runge-Kutta stages (the strong-stability-preserving third-order scheme).  A stage is
//   primitives   per cell: Q -> W = (u, v, P) and T (Newton on the energy, from the cell's previous
//                T), with P from Dalton's law (Sec. 2, Eq. dalton); rho_s are primitives already;
//   fluxes       per face: MP5 left and right states of every primitive variable (Sec. 3.1,
//                Eq. mp5) with the monotonicity-preserving bound (Eqs. mp, ump), and the HLLE
//                flux between them (Eq. fluxhlle);
//   update       per cell: the stage's combination of the sweep's start state, the stage state
//                and dt times the flux difference.
// Up to 16 species one kernel does a stage: a cell's two fluxes, its update and the primitives of
// its new state stay in registers (fluid_stage_x_kernel, fluid_stage_y_kernel), and only the step's
// first primitives have a kernel of their own.  Larger mixtures do a stage in two kernels, with the
// fluxes in memory.  One thread per cell or face; consecutive threads take consecutive x, so every
// array access of a wavefront is one or two contiguous runs of a row.  The six-cell stencil is read
// from the state and primitive arrays, which neighbouring threads share through the caches.
//
// What bounds it: a fused stage of nine species on 1024 x 1024 cells takes 113 us along x and 143 us
// along y, where its 352 bytes a cell at the rate of a large copy (4.7 TB/s) would take 79 us; two
// wavefronts per SIMD (about 210 and 240 registers: the six-cell loads of nine species in flight)
// hide the rest of the latency incompletely, and a bound on the registers makes the compiler spill
// (2.8 ms a step with three wavefronts).  A step takes 1.58 ms; 1.93 ms with the fluxes in memory (a
// stage's faces 58-82 us, its update with primitives 73-100 us), 2.33 ms when also each limiter had a
// division and branches, every coefficient was selected per lane and the energies were summed species
// by species.  3750 cells: 135 us, 182 us and 323 us, of which the fused form saves launches and the
// update its test on a0 per variable, which put each variable's loads behind the last one's.
// 100250 cells of 36 species: 0.93 ms, from 2.22 ms whose Newton summed over the species in every
// iteration.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "kin_internal.h"
#include "kin_xlane.h"

namespace kin {
namespace {

constexpr double kAlphaMP = 2.0;
// Mixtures of at most this many species run kernels compiled for their species count: face states
// and densities stay in registers, and the species loops unroll without a test between them, so the
// loads of one species are not held back until the previous one is done.  Larger mixtures stream
// their species (NSR = 0).
constexpr int kFluidNsRegs = 16;

// median(0, a, b): zero when the signs differ, else the argument of smaller magnitude
__device__ __forceinline__ double minmod(double a, double b) { return fmax(fmin(a, b), fmin(fmax(a, b), 0.0)); }

// Left state of the face j + 1/2 from cells j-2..j+2 (Eq. mp5), limited by the median with u_j
// and u_j + minmod(u_{j+1} - u_j, alpha (u_j - u_{j-1})) (Eqs. mp, ump); the right state is the
// same function of the mirrored stencil.  The bound is itself a median, of u_j, u_{j+1} and
// u_j + alpha (u_j - u_{j-1}), so the whole limiter is minima and maxima: 18 FP64 instructions
// and no division (the branching form with a division by 60 took about 40).  A value that is not
// a number in any of the five cells reaches the result through uL.
__device__ __forceinline__ double mp5(double um2, double um1, double u0, double up1, double up2)
{
    const double uL = fma(up2, -3.0 / 60.0, fma(up1, 27.0 / 60.0, fma(u0, 47.0 / 60.0, fma(um1, -13.0 / 60.0, um2 * (2.0 / 60.0)))));
    const double far = fma(kAlphaMP, u0 - um1, u0);
    const double ump = fmax(fmin(u0, up1), fmin(fmax(u0, up1), far));
    return uL + minmod(u0 - uL, ump - uL);
}

// 1/x from the hardware reciprocal refined by two Newton steps (within an ulp for normal x)
__device__ __forceinline__ double recip(double x)
{
    double y = __builtin_amdgcn_rcp(x);
    y = fma(y, fma(-x, y, 1.0), y);
    return fma(y, fma(-x, y, 1.0), y);
}

struct Grid {
    int ns, nx, ny, bc;   // bc: 0 periodic, 1 zero-gradient
    long long n;          // nx * ny
};

// Byte offset of a cell in an array.  The kernels of a compiled species count use 32 bits (a grid whose
// arrays reach 4 GiB each takes the streamed ones): an access is then a scalar base, which holds the
// variable, and one offset register for all of a cell's variables, instead of a 64-bit address each.
template <int NSR> using Off = std::conditional_t<(NSR > 0), unsigned, unsigned long long>;
template <typename O>
__device__ __forceinline__ double ld(const double *base, O off)
{
    return *reinterpret_cast<const double *>(reinterpret_cast<const char *>(base) + off);
}
template <typename O>
__device__ __forceinline__ void st(double *base, O off, double v)
{
    *reinterpret_cast<double *>(reinterpret_cast<char *>(base) + off) = v;
}

// body(s) for every species: unrolled for a compile-time count, else a loop of four at a time
template <int NSR, typename Body>
__device__ __forceinline__ void each_species(int ns, Body body)
{
    if constexpr (NSR > 0) {
#pragma unroll
        for (int s = 0; s < NSR; ++s) body(s);
    } else {
#pragma unroll 4
        for (int s = 0; s < ns; ++s) body(s);
    }
}

// Coefficients of the mixture's energy as a polynomial in T: with each species' energy
// e_s(T) = sum_k E_sk T^k (fluid table), B_k = sum_s rho_s E_sk gives sum_s rho_s e_s = sum B_k T^k
// and rho c_v = sum k B_k T^(k-1), for one choice of NASA-7 range per species.  The species index
// is uniform, so the coefficients come through scalar loads; a wavefront whose lanes all lie above
// (or all below) every species' switch temperature reads one range and selects nothing.
// Species s has row row(s) of the table.
template <int NSR, typename Dens, typename Row>
__device__ __forceinline__ void mix_coefs(const WaveTables &t, int ns, double T, Dens dens, Row row, double (&B)[6])
{
#pragma unroll
    for (int k = 0; k < 6; ++k) B[k] = 0.0;
    auto one_range = [&](int o, auto share) {   // o = 0 or 6
        // a pointer of its own in each path: the compiler would load what two paths share before the
        // branch, and hold a hundred coefficients in registers across it
        const double *p = t.fl;
        asm volatile("" : "+s"(p));
        const auto *fl = uniform_table(p);
        each_species<NSR>(ns, [&](int s) {
            const double r = share(s, dens(s));
#pragma unroll
            for (int k = 0; k < 6; ++k) B[k] = fma(r, fl[kFluidTab * row(s) + o + k], B[k]);
        });
    };
    auto all = [](int, double r) { return r; };
    const int mode = __builtin_amdgcn_readfirstlane(__all(T >= t.Tsw_hi) ? 2 : (__all(T < t.Tsw_lo) ? 0 : 1));
    if (mode != 1) {
        one_range(3 * mode, all);
    } else {
        // each range with the densities of the species that it holds for (a selection of coefficients would
        // become a load per lane), one range after the other
        const auto *sw = uniform_table(t.fl) + 13;
        one_range(0, [&](int s, double r) { return T < sw[kFluidTab * row(s)] ? r : 0.0; });
        one_range(6, [&](int s, double r) { return T < sw[kFluidTab * row(s)] ? 0.0 : r; });
    }
}

template <int NSR, typename Dens>
__device__ __forceinline__ void mix_coefs(const WaveTables &t, int ns, double T, Dens dens, double (&B)[6])
{
    mix_coefs<NSR>(t, ns, T, dens, [](int s) { return s; }, B);
}

__device__ __forceinline__ double mix_energy(const double (&B)[6], double T)
{
    return fma(T, fma(T, fma(T, fma(T, fma(T, B[5], B[4]), B[3]), B[2]), B[1]), B[0]);
}

__device__ __forceinline__ double mix_cv(const double (&B)[6], double T)
{
    return fma(T, fma(T, fma(T, fma(T, 5.0 * B[5], 4.0 * B[4]), 3.0 * B[3]), 2.0 * B[2]), B[1]);
}

// The temperatures lo <= T' < hi at which every species has the NASA-7 range that it has at T
template <int NSR>
__device__ __forceinline__ void range_interval(const WaveTables &t, int ns, double T, double &lo, double &hi)
{
    lo = -__builtin_inf();
    hi = __builtin_inf();
    if (T >= t.Tsw_hi) {
        lo = t.Tsw_hi;
    } else if (T < t.Tsw_lo) {
        hi = t.Tsw_lo;
    } else {
        const auto *fl = uniform_table(t.fl);
        each_species<NSR>(ns, [&](int s) {
            const double m = fl[kFluidTab * s + 13];
            if (T < m) hi = fmin(hi, m);
            else lo = fmax(lo, m);
        });
    }
}

// Primitive variables of cell i from its conserved state q (ns partial densities, two momenta,
// E; q(v) returns variable v): u, v, P = rho R T into the three rows of W and T into Tc, by
// Newton on the sensible energy from the cell's previous T.  The partial densities are primitives
// as they are, so the face kernel reads them from the state itself.
// Within one choice of NASA-7 range per species the mixture's energy is a polynomial, whose
// coefficients are summed once per choice: an iteration evaluates one polynomial, and the sums are
// redone only when T leaves the interval between switch temperatures that they hold for.
template <int NSR, typename QV>
__device__ __forceinline__ void cell_primitives(const WaveTables &t, const Grid &g, Off<NSR> o, QV q, double *W,
                                                double *Tc)
{
    const int ns = NSR > 0 ? NSR : g.ns;
    const long long n = g.n;
    const auto *fl = uniform_table(t.fl);
    double rho = 0.0, rR = 0.0;
    each_species<NSR>(ns, [&](int s) {
        const double r = q(s);
        rho += r;
        rR = fma(r, fl[kFluidTab * s + 12], rR);
    });
    const double ir = 1.0 / rho;
    const double u = q(ns) * ir, v = q(ns + 1) * ir;
    const double eint = q(ns + 2) - 0.5 * rho * (u * u + v * v);
    double T = ld(Tc, o);
    if (!(T >= 100.0 && T <= 1e4)) T = 1000.0;
    double B[6];
    double lo = 1.0, hi = 0.0;   // B holds for lo <= T < hi (at first for nothing)
    bool go = true;
    for (int it = 0; it < 60 && go; ++it) {
        if (!(T >= lo && T < hi)) {
            mix_coefs<NSR>(t, ns, T, q, B);
            range_interval<NSR>(t, ns, T, lo, hi);
        }
        const double dT = (mix_energy(B, T) - eint) * recip(mix_cv(B, T));
        T -= dT;
        go = fabs(dT) > 1e-13 * fabs(T);   // until converged, or not a number
    }
    st(Tc, o, T);
    st(W, o, u);
    st(W + n, o, v);
    st(W + 2 * n, o, rR * T);
}

template <int NSR>
__global__ void __launch_bounds__(256) fluid_prim_kernel(WaveTables t, Grid g, const double *Q, double *W, double *Tc)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= g.n) return;
    const long long n = g.n;
    if constexpr (NSR > 0) {
        const Off<NSR> o = 8u * (unsigned)i;
        double q[NSR + 3];
#pragma unroll
        for (int v = 0; v < NSR + 3; ++v) q[v] = ld(Q + (size_t)v * n, o);
        cell_primitives<NSR>(t, g, o, [&](int v) { return q[v]; }, W, Tc);
    } else {
        cell_primitives<0>(t, g, 8ull * i, [&](int v) { return Q[(size_t)v * n + i]; }, W, Tc);
    }
}

// Cell index along the sweep direction k (0..len-1 after the boundary rule) of an offset one.
__device__ __forceinline__ int wrap(int k, int len, int bc)
{
    if (bc == 0) return k < 0 ? k + len : (k >= len ? k - len : k);
    return k < 0 ? 0 : (k >= len ? len - 1 : k);
}

// sqrt of a positive number from the hardware's reciprocal square root and two coupled Newton
// steps (within an ulp), zero for zero
__device__ __forceinline__ double sqrt_pos(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    g = fma(fma(-g, g, x), h, g);
    return x == 0.0 ? 0.0 : g;
}

// The HLLE flux of a variable is, with w_L = b+ / (b+ - b-), w_R = -b- / (b+ - b-) and
// p = b+ b- / (b+ - b-), w_L F_L + w_R F_R + p (Q_R - Q_L); every F is Q u_n plus a pressure term,
// so each variable's flux is Q_L (w_L u_L - p) + Q_R (w_R u_R + p) and the pressure's share.
struct Hlle {
    double aL, aR, un, ut, E;   // a species' flux is its L aL + R aR; fluxes of momentum and energy
};

// From the states' velocities, pressures, densities, gas constants rho R, energies and heat capacities.
__device__ __forceinline__ Hlle hlle(double unL, double unR, double utL, double utR, double PL, double PR, double rL, double rR,
                                     double GL, double GR, double eL, double eR, double cvL, double cvR)
{
    const double EL = eL + 0.5 * rL * (unL * unL + utL * utL);
    const double ER = eR + 0.5 * rR * (unR * unR + utR * utR);
    const double c2L = (cvL + GL) * PL * recip(cvL * rL), c2R = (cvR + GR) * PR * recip(cvR * rR);
    const double cL = sqrt_pos(c2L), cR = sqrt_pos(c2R);
    const double sL = sqrt_pos(rL), sR = sqrt_pos(rR);
    const double is = recip(sL + sR), du = unR - unL;
    const double uh = (sL * unL + sR * unR) * is;
    const double c2h = (sL * c2L + sR * c2R) * is + 0.5 * (sL * is) * (sR * is) * (du * du);
    const double ch = sqrt_pos(c2h);
    const double bp = fmax(0.0, fmax(uh + ch, unR + cR));
    const double bm = fmin(0.0, fmin(uh - ch, unL - cL));
    const double idb = recip(bp - bm);
    const double wL = bp * idb, wR = -bm * idb, pm = wL * bm;
    const double aL = fma(wL, unL, -pm), aR = fma(wR, unR, pm);
    const double pP = fma(wL, PL, wR * PR);
    const double mL = rL * aL, mR = rR * aR;
    return {aL, aR, fma(mL, unL, fma(mR, unR, pP)), fma(mL, utL, mR * utR),
            fma(EL, aL, fma(ER, aR, fma(wL * unL, PL, wR * unR * PR)))};
}

// Face fluxes of a sweep along x (DIR 0) or y (DIR 1).  Face a along the sweep lies between
// cells a - 1 and a.  put(v, F) receives the flux of variable v.
// NSR > 0: each species is reconstructed once and both of its states stay in registers; NSR = 0
// reconstructs it again in each pass over the species (three, or two where every species has one
// NASA-7 range, whose energies do not wait for the temperature).
template <int DIR, int NSR, typename Put>
__device__ __forceinline__ void face_flux(const WaveTables &t, const Grid &g, int fx, int fy, const double *Qs,
                                          const double *W, Put put)
{
    const int a = DIR == 0 ? fx : fy;                 // face index along the sweep
    const int len = DIR == 0 ? g.nx : g.ny;
    const long long n = g.n;
    const int ns = NSR > 0 ? NSR : g.ns;
    // cells a-3 .. a+2 along the sweep (j = a - 1 is the face's left cell)
    Off<NSR> c[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const int q = wrap(a - 3 + k, len, g.bc);
        c[k] = 8 * (DIR == 0 ? (Off<NSR>)fy * g.nx + q : (Off<NSR>)q * g.nx + fx);
    }
    auto recon = [&](const double *w, double &L, double &R) {
        const double v0 = ld(w, c[0]), v1 = ld(w, c[1]), v2 = ld(w, c[2]), v3 = ld(w, c[3]), v4 = ld(w, c[4]), v5 = ld(w, c[5]);
        L = mp5(v0, v1, v2, v3, v4);
        R = mp5(v5, v4, v3, v2, v1);
    };
    const double *Wun = W + (size_t)(DIR == 0 ? 0 : 1) * n;
    const double *Wut = W + (size_t)(DIR == 0 ? 1 : 0) * n;
    double unL, unR, utL, utR, PL, PR;
    recon(Wun, unL, unR);
    recon(Wut, utL, utR);
    recon(W + (size_t)2 * n, PL, PR);
    double Ls[NSR > 0 ? NSR : 1], Rv[NSR > 0 ? NSR : 1];
    if constexpr (NSR > 0) {
#pragma unroll
        for (int s = 0; s < NSR; ++s) recon(Qs + (size_t)s * n, Ls[s], Rv[s]);
    }
    auto state = [&](int s, double &L, double &R) {
        if constexpr (NSR > 0) {
            L = Ls[s];
            R = Rv[s];
        } else {
            recon(Qs + (size_t)s * n, L, R);
        }
    };
    // densities, gas constants and temperatures of the two states, then their energies and heat
    // capacities (one side after the other: six coefficients are live at a time)
    const auto *fl = uniform_table(t.fl);
    double rL = 0.0, rR = 0.0, GL = 0.0, GR = 0.0, BL[6], BR[6], TL, TR;
    if constexpr (NSR > 0) {
        each_species<NSR>(ns, [&](int s) {
            const double Rs = fl[kFluidTab * s + 12];
            rL += Ls[s];
            rR += Rv[s];
            GL = fma(Ls[s], Rs, GL);
            GR = fma(Rv[s], Rs, GR);
        });
        TL = PL * recip(GL);
        TR = PR * recip(GR);
        mix_coefs<NSR>(t, ns, TL, [&](int s) { return Ls[s]; }, BL);
    } else {
        const bool one = t.Tsw_hi <= 0.0;   // one range for every species
#pragma unroll
        for (int k = 0; k < 6; ++k) BL[k] = BR[k] = 0.0;
        auto add = [&](int s, double L, double R, bool loL, bool loR) {
            const double Ll = loL ? L : 0.0, Lh = loL ? 0.0 : L, Rl = loR ? R : 0.0, Rh = loR ? 0.0 : R;
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                const double lo = fl[kFluidTab * s + k], hi = fl[kFluidTab * s + 6 + k];
                BL[k] = fma(Ll, lo, fma(Lh, hi, BL[k]));
                BR[k] = fma(Rl, lo, fma(Rh, hi, BR[k]));
            }
        };
        auto add_hi = [&](int s, double L, double R) {
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                BL[k] = fma(L, fl[kFluidTab * s + 6 + k], BL[k]);
                BR[k] = fma(R, fl[kFluidTab * s + 6 + k], BR[k]);
            }
        };
        auto sums = [&](auto with_energy) {
            each_species<0>(ns, [&](int s) {
                double L, R;
                state(s, L, R);
                const double Rs = fl[kFluidTab * s + 12];
                rL += L;
                rR += R;
                GL = fma(L, Rs, GL);
                GR = fma(R, Rs, GR);
                if constexpr (decltype(with_energy)::value) add_hi(s, L, R);
            });
        };
        if (one) sums(std::true_type{});
        else sums(std::false_type{});
        TL = PL * recip(GL);
        TR = PR * recip(GR);
        if (!one)
            each_species<0>(ns, [&](int s) {
                double L, R;
                state(s, L, R);
                const double m = fl[kFluidTab * s + 13];
                add(s, L, R, TL < m, TR < m);
            });
    }
    const double eL = mix_energy(BL, TL), cvL = mix_cv(BL, TL);
    if constexpr (NSR > 0) mix_coefs<NSR>(t, ns, TR, [&](int s) { return Rv[s]; }, BR);
    const double eR = mix_energy(BR, TR), cvR = mix_cv(BR, TR);
    const Hlle h = hlle(unL, unR, utL, utR, PL, PR, rL, rR, GL, GR, eL, eR, cvL, cvR);
    each_species<NSR>(ns, [&](int s) {
        double L, R;
        state(s, L, R);
        put(s, fma(L, h.aL, R * h.aR));
    });
    put(DIR == 0 ? ns : ns + 1, h.un);
    put(DIR == 0 ? ns + 1 : ns, h.ut);
    put(ns + 2, h.E);
}

// Faces are stored [var][ny][nx + 1] (x) or [var][ny + 1][nx] (y).
template <int DIR>
__global__ void __launch_bounds__(256) fluid_flux_kernel(WaveTables t, Grid g, const double *Qs, const double *W, double *F)
{
    const long long f = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const int fw = DIR == 0 ? g.nx + 1 : g.nx;      // faces per row of the face array
    const int fh = DIR == 0 ? g.ny : g.ny + 1;
    const long long fn = (long long)fw * fh;
    if (f >= fn) return;
    face_flux<DIR, 0>(t, g, (int)(f % fw), (int)(f / fw), Qs, W, [&](int v, double x) { F[(size_t)v * fn + f] = x; });
}

// Qout = a0 Q0 + a1 (Q + dt L), L = -(F_{a+1} - F_a) / h (in place allowed: each thread reads
// and writes only its own cell).  r = dt / h.  The variables go in groups whose loads are all issued
// before a store, which the compiler could not move them across; PRIM: then the primitives of the new
// state for the next stage.
template <int DIR, bool PRIM>
__global__ void __launch_bounds__(256) fluid_update_kernel(WaveTables t, Grid g, const double *Q0, const double *Q,
                                                           double *Qout, const double *F, double r, double a0,
                                                           double a1, double *W, double *Tc)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= g.n) return;
    const int x = (int)(i % g.nx), y = (int)(i / g.nx);
    const long long fn = DIR == 0 ? (long long)(g.nx + 1) * g.ny : (long long)g.nx * (g.ny + 1);
    const long long fl = DIR == 0 ? (long long)y * (g.nx + 1) + x : i;
    const long long fr = DIR == 0 ? fl + 1 : fl + g.nx;
    const long long n = g.n;
    const int nv = g.ns + 3;
    constexpr int kGroup = 8;
    for (int v0 = 0; v0 < nv; v0 += kGroup) {
        double dF[kGroup], q[kGroup], q0[kGroup];
#pragma unroll
        for (int k = 0; k < kGroup; ++k) {
            const size_t v = v0 + k < nv ? v0 + k : nv - 1;
            dF[k] = F[v * fn + fl] - F[v * fn + fr];
            q[k] = Q[v * n + i];
            q0[k] = Q0[v * n + i];
        }
#pragma unroll
        for (int k = 0; k < kGroup; ++k)
            if (v0 + k < nv) Qout[(size_t)(v0 + k) * n + i] = fma(a0, q0[k], a1 * fma(r, dF[k], q[k]));
    }
    if constexpr (PRIM) cell_primitives<0>(t, g, 8ull * i, [&](int v) { return Qout[(size_t)v * n + i]; }, W, Tc);
}

// One stage of a sweep in one kernel: the faces of its input, and the update from them in registers, so
// that no flux goes through memory.  Qout = a0 Q0 + a1 (Q + dt L) as in fluid_update_kernel; PRIM also
// forms the primitives of Qout.  The input is read at neighbouring cells, so the output is another array,
// and its primitives go to another set of rows (Wout) than the input's (Win).
template <int NSR, bool PRIM>
__device__ __forceinline__ void stage_update(const WaveTables &t, const Grid &g, Off<NSR> o, const double (&Fl)[NSR + 3],
                                             const double (&Fr)[NSR + 3], const double *Q0, const double *Q, double *Qout,
                                             double r, double a0, double a1, double *Wout, double *Tc)
{
    // (the first stage, a0 = 0, has Q0 = Q: no test stands between the loads)
    double qn[NSR + 3], q0[NSR + 3];
#pragma unroll
    for (int v = 0; v < NSR + 3; ++v) {
        qn[v] = ld(Q + (size_t)v * g.n, o);
        q0[v] = ld(Q0 + (size_t)v * g.n, o);
    }
#pragma unroll
    for (int v = 0; v < NSR + 3; ++v) {
        qn[v] = fma(a0, q0[v], a1 * fma(r, Fl[v] - Fr[v], qn[v]));
        st(Qout + (size_t)v * g.n, o, qn[v]);
    }
    if constexpr (PRIM) cell_primitives<NSR>(t, g, o, [&](int v) { return qn[v]; }, Wout, Tc);
}

// Along x a wavefront takes 64 consecutive faces of the rows laid end to end (nx + 1 a row) and updates
// the cells right of the first 63; a cell's other face comes from the next lane.  No barrier, and one face
// in 64 is computed twice.
template <int NSR, bool PRIM>
__global__ void __launch_bounds__(256) fluid_stage_x_kernel(WaveTables t, Grid g, const double *Q0, const double *Q,
                                                            double *Qout, const double *Win, double *Wout, double *Tc,
                                                            double r, double a0, double a1)
{
    const int lane = threadIdx.x & 63;
    const long long f = ((long long)blockIdx.x * 4 + (threadIdx.x >> 6)) * 63 + lane;
    const int fw = g.nx + 1;
    const long long nf = (long long)fw * g.ny, fc = f < nf ? f : nf - 1;   // every lane computes a face
    const int fx = (int)(fc % fw), fy = (int)(fc / fw);
    double F[NSR + 3], Fr[NSR + 3];
    face_flux<0, NSR>(t, g, fx, fy, Q, Win, [&](int v, double x) { F[v] = x; });
#pragma unroll
    for (int v = 0; v < NSR + 3; ++v) Fr[v] = __shfl_down(F[v], 1);
    if (lane < 63 && f < nf && fx < g.nx)
        stage_update<NSR, PRIM>(t, g, 8u * ((unsigned)fy * g.nx + fx), F, Fr, Q0, Q, Qout, r, a0, a1, Wout, Tc);
}

// Along y a thread walks up `rows` cells of one column, face by face, and keeps the flux of the face
// below; the first face of a run is the last one of the run underneath, computed by both.
template <int NSR, bool PRIM>
__global__ void __launch_bounds__(256) fluid_stage_y_kernel(WaveTables t, Grid g, const double *Q0, const double *Q,
                                                            double *Qout, const double *Win, double *Wout, double *Tc,
                                                            double r, double a0, double a1, int rows)
{
    const long long k = (long long)blockIdx.x * 256 + threadIdx.x;
    const int x = (int)(k % g.nx);
    const long long y0 = k / g.nx * rows;
    if (y0 >= g.ny) return;
    const int y1 = (int)(y0 + rows < g.ny ? y0 + rows : g.ny);
    double F[NSR + 3], Fr[NSR + 3];
    face_flux<1, NSR>(t, g, x, (int)y0, Q, Win, [&](int v, double q) { F[v] = q; });
#pragma unroll 1
    for (int y = (int)y0; y < y1; ++y) {
        face_flux<1, NSR>(t, g, x, y + 1, Q, Win, [&](int v, double q) { Fr[v] = q; });
        stage_update<NSR, PRIM>(t, g, 8u * ((unsigned)y * g.nx + x), F, Fr, Q0, Q, Qout, r, a0, a1, Wout, Tc);
#pragma unroll
        for (int v = 0; v < NSR + 3; ++v) F[v] = Fr[v];
    }
}

// Largest (|u| + c) / dx and (|v| + c) / dy over the grid (positive doubles order like their
// bit patterns, so an unsigned 64-bit atomic maximum finds it).  A block strides over the grid
// and reduces its cells first, so the one word takes one atomic per block, not per wavefront.
constexpr int kSpeedThreads = 256;
constexpr int kSpeedBlocks = 1024;

__global__ void __launch_bounds__(kSpeedThreads) fluid_speed_kernel(WaveTables t, Grid g, const double *Q,
                                                                    const double *W, const double *Tc, double dx,
                                                                    double dy, unsigned long long *out)
{
    __shared__ double wmax[kSpeedThreads / 64];
    double r = 0.0;
    for (long long i = (long long)blockIdx.x * kSpeedThreads + threadIdx.x; i < g.n;
         i += (long long)gridDim.x * kSpeedThreads) {
        const long long n = g.n;
        double rho = 0.0, rR = 0.0, B[6];
        const double T = Tc[i];
        const auto *fl = uniform_table(t.fl);
        mix_coefs<0>(t, g.ns, T, [&](int s) { return Q[(size_t)s * n + i]; }, B);
        for (int s = 0; s < g.ns; ++s) {
            const double rs = Q[(size_t)s * n + i];
            rho += rs;
            rR = fma(rs, fl[kFluidTab * s + 12], rR);
        }
        const double cv = mix_cv(B, T);
        const double P = W[(size_t)2 * n + i];
        const double c = sqrt((cv + rR) / cv * P / rho);
        double ri = fmax((fabs(W[i]) + c) / dx, (fabs(W[(size_t)n + i]) + c) / dy);
        if (!(ri >= 0.0)) ri = __builtin_inf();   // a bad cell makes the step size zero
        r = fmax(r, ri);
    }
    for (int o = 32; o > 0; o >>= 1) r = fmax(r, __shfl_xor(r, o));
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = r;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kSpeedThreads / 64; ++w) r = fmax(r, wmax[w]);
        atomicMax(out, (unsigned long long)__double_as_longlong(r));
    }
}

// Kinetic energy of each cell (kept for the way back), and E - KE, the energy the chemistry
// sub-step sees; after it, E = E_sens + KE with the same KE (chemistry changes neither the
// density nor the momentum).
__global__ void fluid_kinetic_kernel(Grid g, const double *Q, double *KE, double *Es)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= g.n) return;
    const long long n = g.n;
    double rho = 0.0;
    for (int s = 0; s < g.ns; ++s) rho += Q[(size_t)s * n + i];
    const double mx = Q[(size_t)g.ns * n + i], my = Q[(size_t)(g.ns + 1) * n + i];
    const double ke = 0.5 * (mx * mx + my * my) / rho;
    KE[i] = ke;
    Es[i] = Q[(size_t)(g.ns + 2) * n + i] - ke;
}

__global__ void fluid_energy_back_kernel(Grid g, double *Q, const double *KE, const double *Es)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= g.n) return;
    Q[(size_t)(g.ns + 2) * g.n + i] = Es[i] + KE[i];
}

// f(std::integral_constant<int, NSR>): the species count itself up to kFluidNsRegs, else (or where 32-bit
// offsets do not reach) 0, the streamed kernels
template <int NSR = 1, typename Fn>
void ns_class(const Grid &g, Fn f)
{
    if constexpr (NSR > kFluidNsRegs) f(std::integral_constant<int, 0>{});
    else if (g.ns == NSR && g.n < (1ll << 29)) f(std::integral_constant<int, NSR>{});
    else ns_class<NSR + 1>(g, f);
}

}  // namespace

// Rows that a thread of the y stage walks: its first face is extra work, so as many as leave the device
// two wavefronts per SIMD (2048), at most kMaxRows
constexpr int kMaxRows = 8;
static int rows_per_thread(const Grid &g)
{
    const long long r = g.n / (2048 * 64);
    return r < 1 ? 1 : (r > kMaxRows ? kMaxRows : (int)r);
}

hipError_t launch_fluid_step(const WaveTables &t, const FluidGrid &fg, double dt, double dx, double dy, bool y_first,
                             double *Q, double *Q1, double *W, double *T, double *F, hipStream_t s)
{
    const Grid g{t.ns, fg.nx, fg.ny, fg.bc, (long long)fg.nx * fg.ny};
    const int block = 256;
    const unsigned gc = (unsigned)((g.n + block - 1) / block);
    // (a0, a1, stage input, stage output): Q1 = Q + dt L(Q); Q2 = 3/4 Q + 1/4 (Q1 + dt L(Q1));
    // Q <- 1/3 Q + 2/3 (Q2 + dt L(Q2))
    const double a0[3] = {0.0, 0.75, 1.0 / 3.0}, a1[3] = {1.0, 0.25, 2.0 / 3.0};
    ns_class(g, [&](auto nsrc) {
        constexpr int NSR = decltype(nsrc)::value;
        if constexpr (NSR > 0) {
            // Q2 takes the place of the fluxes; the primitives alternate between two sets of rows
            double *const buf[3] = {Q, Q1, F}, *const prim[2] = {W, W + (size_t)3 * g.n};
            hipLaunchKernelGGL((fluid_prim_kernel<NSR>), dim3(gc), dim3(block), 0, s, t, g, Q, prim[0], T);
            int w = 0;
            for (int sweep = 0; sweep < 2; ++sweep) {
                const bool along_x = (sweep == 0) != y_first;
                const double r = dt / (along_x ? dx : dy);
                for (int k = 0; k < 3; ++k, w ^= 1) {
                    const double *in = buf[k];
                    double *out = buf[(k + 1) % 3];
                    const bool last = sweep == 1 && k == 2;   // no stage reads its primitives
                    if (along_x) {
                        const long long waves = ((long long)(g.nx + 1) * g.ny + 62) / 63;
                        const unsigned gx = (unsigned)((waves + 3) / 4);
                        if (last)
                            hipLaunchKernelGGL((fluid_stage_x_kernel<NSR, false>), dim3(gx), dim3(block), 0, s, t, g, Q, in, out,
                                               prim[w], prim[w ^ 1], T, r, a0[k], a1[k]);
                        else
                            hipLaunchKernelGGL((fluid_stage_x_kernel<NSR, true>), dim3(gx), dim3(block), 0, s, t, g, Q, in, out,
                                               prim[w], prim[w ^ 1], T, r, a0[k], a1[k]);
                    } else {
                        const int rows = rows_per_thread(g);
                        const long long threads = (long long)g.nx * ((g.ny + rows - 1) / rows);
                        const unsigned gy = (unsigned)((threads + block - 1) / block);
                        if (last)
                            hipLaunchKernelGGL((fluid_stage_y_kernel<NSR, false>), dim3(gy), dim3(block), 0, s, t, g, Q, in, out,
                                               prim[w], prim[w ^ 1], T, r, a0[k], a1[k], rows);
                        else
                            hipLaunchKernelGGL((fluid_stage_y_kernel<NSR, true>), dim3(gy), dim3(block), 0, s, t, g, Q, in, out,
                                               prim[w], prim[w ^ 1], T, r, a0[k], a1[k], rows);
                    }
                }
            }
        } else {
            // larger mixtures: a stage is its faces' kernel, then the update's, which in the first two
            // stages also forms the primitives of its output
            auto sweep = [&](auto dirc) {
                constexpr int D = decltype(dirc)::value;
                const long long nf = D == 0 ? (long long)(g.nx + 1) * g.ny : (long long)g.nx * (g.ny + 1);
                const unsigned gf = (unsigned)((nf + block - 1) / block);
                const double r = dt / (D == 0 ? dx : dy);
                hipLaunchKernelGGL((fluid_prim_kernel<0>), dim3(gc), dim3(block), 0, s, t, g, Q, W, T);
                for (int k = 0; k < 3; ++k) {
                    const double *in = k == 0 ? Q : Q1;
                    hipLaunchKernelGGL((fluid_flux_kernel<D>), dim3(gf), dim3(block), 0, s, t, g, in, W, F);
                    if (k == 2)
                        hipLaunchKernelGGL((fluid_update_kernel<D, false>), dim3(gc), dim3(block), 0, s, t, g, Q, in, Q, F, r,
                                           a0[k], a1[k], W, T);
                    else
                        hipLaunchKernelGGL((fluid_update_kernel<D, true>), dim3(gc), dim3(block), 0, s, t, g, Q, in, Q1, F, r,
                                           a0[k], a1[k], W, T);
                }
            };
            if (y_first) sweep(std::integral_constant<int, 1>{});
            sweep(std::integral_constant<int, 0>{});
            if (!y_first) sweep(std::integral_constant<int, 1>{});
        }
    });
    return hipGetLastError();
}

hipError_t launch_fluid_speed(const WaveTables &t, const FluidGrid &fg, const double *Q, double *W, double *T,
                              double dx, double dy, unsigned long long *out, hipStream_t s)
{
    const Grid g{t.ns, fg.nx, fg.ny, fg.bc, (long long)fg.nx * fg.ny};
    const int block = 256;
    const unsigned gc = (unsigned)((g.n + block - 1) / block);
    ns_class(g, [&](auto nsrc) {
        constexpr int NSR = decltype(nsrc)::value;
        hipLaunchKernelGGL((fluid_prim_kernel<NSR>), dim3(gc), dim3(block), 0, s, t, g, Q, W, T);
    });
    const long long sb = (g.n + kSpeedThreads - 1) / kSpeedThreads;
    hipLaunchKernelGGL(fluid_speed_kernel, dim3((unsigned)(sb < kSpeedBlocks ? sb : kSpeedBlocks)), dim3(kSpeedThreads),
                       0, s, t, g, Q, W, T, dx, dy, out);
    return hipGetLastError();
}

hipError_t launch_fluid_kinetic(const FluidGrid &fg, int ns, const double *Q, double *KE, double *Es, hipStream_t s)
{
    const Grid g{ns, fg.nx, fg.ny, fg.bc, (long long)fg.nx * fg.ny};
    const int block = 256;
    hipLaunchKernelGGL(fluid_kinetic_kernel, dim3((unsigned)((g.n + block - 1) / block)), dim3(block), 0, s, g, Q, KE, Es);
    return hipGetLastError();
}

hipError_t launch_fluid_energy_back(const FluidGrid &fg, int ns, double *Q, const double *KE, const double *Es,
                                    hipStream_t s)
{
    const Grid g{ns, fg.nx, fg.ny, fg.bc, (long long)fg.nx * fg.ny};
    const int block = 256;
    hipLaunchKernelGGL(fluid_energy_back_kernel, dim3((unsigned)((g.n + block - 1) / block)), dim3(block), 0, s, g, Q, KE, Es);
    return hipGetLastError();
}

}  // namespace kin
