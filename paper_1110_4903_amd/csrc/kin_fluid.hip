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
// One kernel does a stage: a cell's two fluxes, its update and the primitives of its new state stay
// in registers, and only the step's first primitives have a kernel of their own.  Up to 9 species a
// lane does all of a face and a cell (fluid_stage_kernel); two wavefronts share them from 10 to 16 species
// (and of 9 on small grids), four from 17 to 64 (fluid_wide_kernel).  Larger mixtures, and grids
// whose arrays exceed 32-bit offsets, do a stage in two kernels, with the fluxes in memory.
// Consecutive lanes take consecutive x, so an access of a wavefront is a few contiguous runs of a
// row.  The six-cell stencil is read from the state and primitive arrays, which neighbouring lanes
// share through the caches.
//
// What bounds it: a stage of nine species on 1024 x 1024 cells takes 102 us along x and 120 us along
// y, where its 352 bytes a cell at the rate of a large copy (4.7 TB/s) would take 79 us.  A wavefront
// waits for loads in 30% of its cycles and for an instruction to issue in 40%, with the VALU active in a
// third of the SIMDs' cycles: too few wavefronts to cover either wait (208 registers, two on a SIMD at
// most, 1.5 on average), and a bound on the registers makes the compiler spill (three wavefronts: 1.8
// times the time).  36 species on 401 x 250 cells: 36 and 41 us, of 34 us of traffic that the caches partly
// hold (waits 30% and 40%, VALU 43%).  3750 cells of nine species: 7 us a stage, one wavefront's latency.
// us a step, 1024 x 1024 of 9 / 75 x 50 of 9 / 401 x 250 of 36 species:
//   1166 / 162 / 1111  a division and branches in each limiter, a selection of every coefficient per
//                      lane, energies summed species by species
//    963 /  91 /  493  without those; three kernels a stage (faces 58-82 us, update with primitives
//                      73-100 us on the large grid)
//    777 /  67 /  468  one kernel a stage up to 16 species, along y a walk up the columns
//    687 /  57 /  247  tiles along y, tiles to XCDs in contiguous parts, the wide form
//    687 /  50 /  240  the wide form of two wavefronts on small grids
//    689 /  50 /  229  lanes without a cell read nothing
#include <hip/hip_runtime.h>

#include <type_traits>

#include "kin_internal.h"
#include "kin_xlane.h"

namespace kin {
namespace {

constexpr double kAlphaMP = 2.0;
// Up to this many species a wavefront's kernels are compiled for their count (the stages of larger mixtures
// for a part of it): face states and densities stay in registers, and the species loops unroll without a
// test between them, so the loads of one species are not held back until the previous one is done.
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

// Faces of a wavefront.  Along x 64 consecutive ones of the rows laid end to end (nx + 1 a row), and the
// cells right of the first 63.  Along y a tile of 2^lw columns by 64 / 2^lw faces and the cells above all
// but the last of each column.  A cell's other face comes from the lane `next` further on: no barrier, and
// one face of a run is computed twice.
struct Tile {
    int fx, fy;     // the lane's face
    int next;
    bool active;    // the lane has a cell
};
// Consecutive blocks go to the eight XCDs in turn, each with an L2 of its own: block b of the grid (a
// multiple of eight) takes a place in one of eight contiguous parts, so that the rows and cache lines that
// neighbouring tiles share are read into one L2.
__device__ __forceinline__ unsigned xcd_block()
{
    return (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
}

template <int DIR>
__device__ __forceinline__ Tile stage_tile(const Grid &g, long long wave, int lane, int lw)
{
    if constexpr (DIR == 0) {
        const long long f = wave * 63 + lane;
        const int fw = g.nx + 1;
        const long long nf = (long long)fw * g.ny, fc = f < nf ? f : nf - 1;   // every lane computes a face
        const int fx = (int)(fc % fw);
        return {fx, (int)(fc / fw), 1, lane < 63 && f < nf && fx < g.nx};
    } else {
        const int width = 1 << lw, height = 64 >> lw, tiles = (g.nx + width - 1) >> lw;
        const int x = (int)(wave % tiles) * width + (lane & (width - 1));
        const long long y = wave / tiles * (height - 1) + (lane >> lw);
        return {x < g.nx ? x : g.nx - 1, (int)(y < g.ny ? y : g.ny), width, (lane >> lw) < height - 1 && x < g.nx && y < g.ny};
    }
}

template <int DIR, int NSR, bool PRIM>
__global__ void __launch_bounds__(256) fluid_stage_kernel(WaveTables t, Grid g, const double *Q0, const double *Q,
                                                          double *Qout, const double *Win, double *Wout, double *Tc,
                                                          double r, double a0, double a1, int lw)
{
    const int lane = threadIdx.x & 63;
    const Tile c = stage_tile<DIR>(g, (long long)xcd_block() * 4 + (threadIdx.x >> 6), lane, lw);
    double F[NSR + 3], Fr[NSR + 3];
    face_flux<DIR, NSR>(t, g, c.fx, c.fy, Q, Win, [&](int v, double x) { F[v] = x; });
#pragma unroll
    for (int v = 0; v < NSR + 3; ++v) Fr[v] = __shfl_down(F[v], c.next);
    if (c.active)
        stage_update<NSR, PRIM>(t, g, 8u * ((unsigned)c.fy * g.nx + c.fx), F, Fr, Q0, Q, Qout, r, a0, a1, Wout, Tc);
}

// ---- A stage of larger mixtures: NW wavefronts work on the same 64 faces (or cells), lane by lane,
// each on its own run of at most NSG species, whose face states stay in its registers; sums over the
// species go through LDS, and every wavefront then evaluates the face's (cell's) scalars for itself.
// LDS of a block, [..][64 lanes].  The arrays of one union alternate: between two writes of it, and
// between a write and the last reads of the other member, lies a barrier of the other union's exchange.
template <int NW> struct WideShared {
    union {
        struct {
            double sum[NW][4][64];    // face: rho and rho R of the left and the right state
            double prim[3][2][64];       // the states of u, v, P
        } f;
        struct {
            double sum[NW][2][64];    // cell: rho and rho R
            double var[3][64];           // momenta and energy
        } c;
    } a;
    union {
        double e[NW][4][64];          // face: energy and heat capacity of both states
        double B[NW][6][64];          // cell: coefficients of the mixture's energy
    } b;
};

// A wavefront's species are s0 .. s0 + NSG - 1; those from ns on are the last species with no density.
template <int NSG, int NW> struct WideRun {
    // Momenta and energy, and likewise u, v and P, are dealt from the last wavefront on, which may have fewer
    // species; from 3 on there is none.
    static constexpr int kExtra = (3 + NW - 1) / NW;
    int w, s0, ns;
    __device__ __forceinline__ int row(int j) const { return s0 + j < ns ? s0 + j : ns - 1; }
    __device__ __forceinline__ bool has(int j) const { return s0 + j < ns; }
    __device__ __forceinline__ int extra(int j) const { return NW - 1 - w + NW * j; }
    __device__ __forceinline__ int extra_row(int j) const { return extra(j) < 3 ? extra(j) : 2; }
};

// Fluxes of the wavefront's species into F[0..NSG-1], of its momenta or energy behind them.
template <int DIR, int NSG, int NW>
__device__ __forceinline__ void face_flux_wide(const WaveTables &t, const Grid &g, const WideRun<NSG, NW> &run, int lane, int fx,
                                               int fy, const double *Qs, const double *W, WideShared<NW> &sh,
                                               double (&F)[NSG + WideRun<NSG, NW>::kExtra])
{
    const int a = DIR == 0 ? fx : fy;
    const int len = DIR == 0 ? g.nx : g.ny;
    const long long n = g.n;
    unsigned c[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const int q = wrap(a - 3 + k, len, g.bc);
        c[k] = 8 * (DIR == 0 ? (unsigned)fy * g.nx + q : (unsigned)q * g.nx + fx);
    }
    auto recon = [&](const double *w, double &L, double &R) {
        const double v0 = ld(w, c[0]), v1 = ld(w, c[1]), v2 = ld(w, c[2]), v3 = ld(w, c[3]), v4 = ld(w, c[4]), v5 = ld(w, c[5]);
        L = mp5(v0, v1, v2, v3, v4);
        R = mp5(v5, v4, v3, v2, v1);
    };
    constexpr int EX = WideRun<NSG, NW>::kExtra;
    double Ls[NSG], Rv[NSG], pl[EX], pr[EX];
#pragma unroll
    for (int j = 0; j < EX; ++j) recon(W + (size_t)run.extra_row(j) * n, pl[j], pr[j]);
#pragma unroll
    for (int j = 0; j < NSG; ++j) {
        recon(Qs + (size_t)run.row(j) * n, Ls[j], Rv[j]);
        if (!run.has(j)) Ls[j] = Rv[j] = 0.0;
    }
    const auto *fl = uniform_table(t.fl);
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
#pragma unroll
    for (int j = 0; j < NSG; ++j) {
        const double Rs = fl[kFluidTab * run.row(j) + 12];
        s0 += Ls[j];
        s1 += Rv[j];
        s2 = fma(Ls[j], Rs, s2);
        s3 = fma(Rv[j], Rs, s3);
    }
    auto &A = sh.a.f;
    A.sum[run.w][0][lane] = s0;
    A.sum[run.w][1][lane] = s1;
    A.sum[run.w][2][lane] = s2;
    A.sum[run.w][3][lane] = s3;
#pragma unroll
    for (int j = 0; j < EX; ++j)
        if (run.extra(j) < 3) {
            A.prim[run.extra(j)][0][lane] = pl[j];
            A.prim[run.extra(j)][1][lane] = pr[j];
        }
    __syncthreads();
    double rL = 0.0, rR = 0.0, GL = 0.0, GR = 0.0;
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        rL += A.sum[k][0][lane];
        rR += A.sum[k][1][lane];
        GL += A.sum[k][2][lane];
        GR += A.sum[k][3][lane];
    }
    const double unL = A.prim[DIR == 0 ? 0 : 1][0][lane], unR = A.prim[DIR == 0 ? 0 : 1][1][lane];
    const double utL = A.prim[DIR == 0 ? 1 : 0][0][lane], utR = A.prim[DIR == 0 ? 1 : 0][1][lane];
    const double PL = A.prim[2][0][lane], PR = A.prim[2][1][lane];
    const double TL = PL * recip(GL), TR = PR * recip(GR);
    auto row = [&](int j) { return run.row(j); };
    double B[6];
    mix_coefs<NSG>(t, NSG, TL, [&](int j) { return Ls[j]; }, row, B);
    sh.b.e[run.w][0][lane] = mix_energy(B, TL);
    sh.b.e[run.w][1][lane] = mix_cv(B, TL);
    mix_coefs<NSG>(t, NSG, TR, [&](int j) { return Rv[j]; }, row, B);
    sh.b.e[run.w][2][lane] = mix_energy(B, TR);
    sh.b.e[run.w][3][lane] = mix_cv(B, TR);
    __syncthreads();
    double eL = 0.0, cvL = 0.0, eR = 0.0, cvR = 0.0;
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        eL += sh.b.e[k][0][lane];
        cvL += sh.b.e[k][1][lane];
        eR += sh.b.e[k][2][lane];
        cvR += sh.b.e[k][3][lane];
    }
    const Hlle h = hlle(unL, unR, utL, utR, PL, PR, rL, rR, GL, GR, eL, eR, cvL, cvR);
#pragma unroll
    for (int j = 0; j < NSG; ++j) F[j] = fma(Ls[j], h.aL, Rv[j] * h.aR);
#pragma unroll
    for (int j = 0; j < EX; ++j)
        F[NSG + j] = run.extra(j) == (DIR == 0 ? 0 : 1) ? h.un : (run.extra(j) == (DIR == 0 ? 1 : 0) ? h.ut : h.E);
}

// stage_update for the wavefront's variables of a cell (active: of the grid, and this lane's), then, with
// PRIM, its primitives: every wavefront iterates on the same sums, and they share the storing of T, u, v and P.
template <int NSG, int NW, bool PRIM>
__device__ __forceinline__ void stage_update_wide(const WaveTables &t, const Grid &g, const WideRun<NSG, NW> &run, int lane,
                                                  bool active, unsigned o, const double (&Fl)[NSG + WideRun<NSG, NW>::kExtra],
                                                  const double (&Fr)[NSG + WideRun<NSG, NW>::kExtra], const double *Q0, const double *Q,
                                                  double *Qout, double r, double a0, double a1, double *W, double *Tc,
                                                  WideShared<NW> &sh)
{
    const long long n = g.n;
    constexpr int EX = WideRun<NSG, NW>::kExtra;
    // Q0 and Tc of a cell belong to the lane that has it (Q0 is Qout in the last stage, and Tc is both read
    // and written): the others read neither, and take an active lane's T so that the wavefront's choice of
    // NASA-7 ranges stays the active lanes' own.
    double qn[NSG + EX], q0[NSG + EX], T = 0.0;
    if (active) {
#pragma unroll
        for (int j = 0; j < NSG + EX; ++j) {
            const size_t v = j < NSG ? run.row(j) : run.ns + run.extra_row(j - NSG);
            qn[j] = ld(Q + v * n, o);
            q0[j] = ld(Q0 + v * n, o);
        }
        if constexpr (PRIM) T = ld(Tc, o);
    } else {
#pragma unroll
        for (int j = 0; j < NSG + EX; ++j) qn[j] = q0[j] = 0.0;
    }
    if constexpr (PRIM) {
        const unsigned long long with = __ballot(active);
        const double Ta = __shfl(T, with ? __builtin_ctzll(with) : 0);
        if (!active) T = Ta;
    }
#pragma unroll
    for (int j = 0; j < NSG + EX; ++j) {
        qn[j] = fma(a0, q0[j], a1 * fma(r, Fl[j] - Fr[j], qn[j]));
        const bool mine = j < NSG ? run.has(j) : run.extra(j - NSG) < 3;
        const size_t v = j < NSG ? run.row(j) : run.ns + run.extra_row(j - NSG);
        if (mine && active) st(Qout + v * n, o, qn[j]);
        if (j < NSG && !mine) qn[j] = 0.0;
    }
    if constexpr (PRIM) {
        const auto *fl = uniform_table(t.fl);
        double s0 = 0.0, s1 = 0.0;
#pragma unroll
        for (int j = 0; j < NSG; ++j) {
            s0 += qn[j];
            s1 = fma(qn[j], fl[kFluidTab * run.row(j) + 12], s1);
        }
        auto &C = sh.a.c;
        C.sum[run.w][0][lane] = s0;
        C.sum[run.w][1][lane] = s1;
#pragma unroll
        for (int j = 0; j < EX; ++j)
            if (run.extra(j) < 3) C.var[run.extra(j)][lane] = qn[NSG + j];
        __syncthreads();
        double rho = 0.0, rR = 0.0;
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            rho += C.sum[k][0][lane];
            rR += C.sum[k][1][lane];
        }
        const double ir = 1.0 / rho;
        const double u = C.var[0][lane] * ir, v = C.var[1][lane] * ir;
        const double eint = C.var[2][lane] - 0.5 * rho * (u * u + v * v);
        if (!(T >= 100.0 && T <= 1e4)) T = 1000.0;
        // the iteration of cell_primitives; the block sums coefficients again while a lane has left the
        // interval that its own hold for (the vote is over the block, so all wavefronts do the same)
        bool go = active;
        int it = 0;
        for (int sums = 0; sums < 60; ++sums) {
            double B[6], lo, hi;
            mix_coefs<NSG>(t, NSG, T, [&](int j) { return qn[j]; }, [&](int j) { return run.row(j); }, B);
#pragma unroll
            for (int k = 0; k < 6; ++k) sh.b.B[run.w][k][lane] = B[k];
            __syncthreads();
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                B[k] = 0.0;
#pragma unroll
                for (int q = 0; q < NW; ++q) B[k] += sh.b.B[q][k][lane];
            }
            range_interval<0>(t, run.ns, T, lo, hi);
            while (go && it < 60 && T >= lo && T < hi) {
                const double dT = (mix_energy(B, T) - eint) * recip(mix_cv(B, T));
                T -= dT;
                go = fabs(dT) > 1e-13 * fabs(T);
                ++it;
            }
            if (!__syncthreads_or(go && it < 60 && T == T)) break;
        }
        if (active) {
            if (run.w == 0) st(Tc, o, T);
#pragma unroll
            for (int j = 0; j < EX; ++j)
                if (run.extra(j) < 3)
                    st(W + (size_t)run.extra(j) * n, o, run.extra(j) == 0 ? u : (run.extra(j) == 1 ? v : rR * T));
        }
    }
}

template <int NSG, int NW> __device__ __forceinline__ WideRun<NSG, NW> wide_run(const Grid &g)
{
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    return {w, w * NSG, g.ns};
}

// fluid_stage_kernel with a block per 64 faces.
template <int DIR, int NSG, int NW, bool PRIM>
__global__ void __launch_bounds__(64 * NW) fluid_wide_kernel(WaveTables t, Grid g, const double *Q0, const double *Q,
                                                                double *Qout, const double *Win, double *Wout, double *Tc,
                                                                double r, double a0, double a1, int lw)
{
    __shared__ WideShared<NW> sh;
    const WideRun<NSG, NW> run = wide_run<NSG, NW>(g);
    constexpr int EX = WideRun<NSG, NW>::kExtra;
    const int lane = threadIdx.x & 63;
    const Tile c = stage_tile<DIR>(g, xcd_block(), lane, lw);
    double F[NSG + EX], Fr[NSG + EX];
    face_flux_wide<DIR, NSG, NW>(t, g, run, lane, c.fx, c.fy, Q, Win, sh, F);
#pragma unroll
    for (int j = 0; j < NSG + EX; ++j) Fr[j] = __shfl_down(F[j], c.next);
    const int x = c.fx < g.nx ? c.fx : g.nx - 1, y = c.fy < g.ny ? c.fy : g.ny - 1;
    stage_update_wide<NSG, NW, PRIM>(t, g, run, lane, c.active, 8u * ((unsigned)y * g.nx + x), F, Fr, Q0, Q, Qout, r, a0, a1, Wout,
                                 Tc, sh);
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

// f(N, NW): up to kFluidNsOne species the kernels compiled for N of them (NW = 1), then (and for that many in
// small grids) up to 16 species those of two wavefronts that take at most N each, up to 64 those of four;
// else (or where 32-bit offsets do not reach) N = 0, the streamed kernels.
// Two wavefronts shorten a face's chain, and do its scalars twice; from 12 species on a lane that does a face
// alone leaves one wavefront on a SIMD (256 registers, 13 species).  us a step with one and with two, on
// 160^2, 512^2 and 1024^2 cells:
//   9 species  55 and 56, 166 and 175,  635 and 651     13 species  69 and 64, 289 and 220, 1188 and 900
//  10 species  58 and 56, 179 and 176,  728 and 703     14 species  73 and 64, 305 and 223, 1279 and 930
//  12 species  65 and 60, 232 and 207,  963 and 824     16 species  79 and 70, 333 and 250, 1404 and 1060
// Nine species on small grids: 3750 cells 54.8 and 47.4, 15000 cells 55.3 and 51.3, 25200 cells 56.6 and 55.6.
constexpr long long kFluidSmall = 16384;
constexpr int kFluidNsOne = 9;
template <int N = 1, typename Fn>
void ns_class(const Grid &g, Fn f)
{
    using std::integral_constant;
    if constexpr (N > kFluidNsRegs) {
        f(integral_constant<int, 0>{}, integral_constant<int, 1>{});
    } else {
        // (four wavefronts are up to 8.2 threads a cell, of which a grid holds less than 2^32)
        const bool reach = g.n < (1ll << 29), reach4 = g.n < (1ll << 32) / 9;
        const bool two = g.ns <= 16 && (g.ns > kFluidNsOne || (g.ns == kFluidNsOne && g.n <= kFluidSmall));
        if constexpr (N <= kFluidNsOne)
            if (reach && !two && g.ns == N) return f(integral_constant<int, N>{}, integral_constant<int, 1>{});
        if constexpr (N >= 5 && N <= 8)
            if (reach && two && (g.ns + 1) / 2 == N) return f(integral_constant<int, N>{}, integral_constant<int, 2>{});
        if constexpr (N >= 5)
            if (reach4 && g.ns > 16 && (g.ns + 3) / 4 == N) return f(integral_constant<int, N>{}, integral_constant<int, 4>{});
        ns_class<N + 1>(g, f);
    }
}

// Primitives of Q by the kernel compiled for the species count, up to 16, or the streamed one.
template <int N = 1>
void launch_prim(const WaveTables &t, const Grid &g, const double *Q, double *W, double *T, hipStream_t s)
{
    if constexpr (N > 16) {
        hipLaunchKernelGGL(fluid_prim_kernel<0>, dim3((unsigned)((g.n + 255) / 256)), dim3(256), 0, s, t, g, Q, W, T);
    } else {
        if (g.ns != N || g.n >= (1ll << 29)) return launch_prim<N + 1>(t, g, Q, W, T, s);
        hipLaunchKernelGGL(fluid_prim_kernel<N>, dim3((unsigned)((g.n + 255) / 256)), dim3(256), 0, s, t, g, Q, W, T);
    }
}

// Width (its logarithm) of a tile of the stages along y, of a grid that is that wide: 8 columns by 8 faces
// compute 8/7 of the faces and read 64 contiguous bytes at a time.  Nine species on 1024 x 1024 cells,
// 36 on 401 x 250, us a step: width 4 774 and 385, 8 687 and 247, 16 693 and 255 (4 without the
// assignment of tiles to XCDs).  A thread that walks 8 rows of a column instead, 777 and 388.
// A grid of fewer than four rows takes wider tiles, whose lanes would else have no cell in seven of eight:
// 262144 x 1 cells of 4, 9, 16 and 20 species, us a step, 8 columns 242, 474, 1043 and 978 (which is also
// 32 lanes a cell, more threads from 2^27 cells on than a grid holds), 32 columns 113, 195, 403 and 394.
constexpr int kTileLog = 3;

// One stage, its input's primitives in Win and its output's to Wout (PRIM).
template <int N, int NW, bool PRIM>
void launch_stage(const WaveTables &t, const Grid &g, bool along_x, const double *Q0, const double *Q, double *Qout,
                  const double *Win, double *Wout, double *T, double r, double a0, double a1, hipStream_t s)
{
    int widest = kTileLog, lw = 0;
    while (widest < 5 && (64 >> (widest + 1)) > g.ny) ++widest;
    while (lw < widest && (1 << lw) < g.nx) ++lw;
    const int height = 64 >> lw;
    const long long waves = along_x ? ((long long)(g.nx + 1) * g.ny + 62) / 63
                                    : (long long)((g.nx + (1 << lw) - 1) >> lw) * ((g.ny + height - 2) / (height - 1));
    const dim3 block(NW > 1 ? 64 * NW : 256), grid((unsigned)(((NW > 1 ? waves : (waves + 3) / 4) + 7) / 8 * 8));
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, block, 0, s, t, g, Q0, Q, Qout, Win, Wout, T, r, a0, a1, lw);
    };
    if constexpr (NW > 1) {
        if (along_x) go(fluid_wide_kernel<0, N, NW, PRIM>);
        else go(fluid_wide_kernel<1, N, NW, PRIM>);
    } else {
        if (along_x) go(fluid_stage_kernel<0, N, PRIM>);
        else go(fluid_stage_kernel<1, N, PRIM>);
    }
}

}  // namespace

hipError_t launch_fluid_step(const WaveTables &t, const FluidGrid &fg, double dt, double dx, double dy, bool y_first,
                             double *Q, double *Q1, double *W, double *T, double *F, hipStream_t s)
{
    const Grid g{t.ns, fg.nx, fg.ny, fg.bc, (long long)fg.nx * fg.ny};
    const int block = 256;
    // (a0, a1, stage input, stage output): Q1 = Q + dt L(Q); Q2 = 3/4 Q + 1/4 (Q1 + dt L(Q1));
    // Q <- 1/3 Q + 2/3 (Q2 + dt L(Q2))
    const double a0[3] = {0.0, 0.75, 1.0 / 3.0}, a1[3] = {1.0, 0.25, 2.0 / 3.0};
    ns_class(g, [&](auto nc, auto nwc) {
        constexpr int N = decltype(nc)::value;
        constexpr int NW = decltype(nwc)::value;
        launch_prim(t, g, Q, W, T, s);
        if constexpr (N > 0) {
            // Q2 takes the place of the fluxes; the primitives alternate between two sets of rows
            double *const buf[3] = {Q, Q1, F}, *const prim[2] = {W, W + (size_t)3 * g.n};
            for (int k = 0; k < 6; ++k) {
                const bool along_x = (k < 3) != y_first;
                const double *in = buf[k % 3];
                double *out = buf[(k + 1) % 3];
                const double r = dt / (along_x ? dx : dy);
                if (k < 5)
                    launch_stage<N, NW, true>(t, g, along_x, Q, in, out, prim[k & 1], prim[~k & 1], T, r, a0[k % 3], a1[k % 3], s);
                else   // no stage reads its primitives
                    launch_stage<N, NW, false>(t, g, along_x, Q, in, out, prim[k & 1], prim[~k & 1], T, r, a0[k % 3], a1[k % 3], s);
            }
        } else {
            // a stage is its faces' kernel, then the update's, which but for the step's last also forms the
            // primitives of its output
            const unsigned gc = (unsigned)((g.n + block - 1) / block);
            auto sweep = [&](auto dirc, bool last_sweep) {
                constexpr int D = decltype(dirc)::value;
                const long long nf = D == 0 ? (long long)(g.nx + 1) * g.ny : (long long)g.nx * (g.ny + 1);
                const unsigned gf = (unsigned)((nf + block - 1) / block);
                const double r = dt / (D == 0 ? dx : dy);
                for (int k = 0; k < 3; ++k) {
                    const double *in = k == 0 ? Q : Q1;
                    double *out = k == 2 ? Q : Q1;
                    hipLaunchKernelGGL((fluid_flux_kernel<D>), dim3(gf), dim3(block), 0, s, t, g, in, W, F);
                    if (k == 2 && last_sweep)
                        hipLaunchKernelGGL((fluid_update_kernel<D, false>), dim3(gc), dim3(block), 0, s, t, g, Q, in, out, F, r,
                                           a0[k], a1[k], W, T);
                    else
                        hipLaunchKernelGGL((fluid_update_kernel<D, true>), dim3(gc), dim3(block), 0, s, t, g, Q, in, out, F, r,
                                           a0[k], a1[k], W, T);
                }
            };
            if (y_first) sweep(std::integral_constant<int, 1>{}, false);
            sweep(std::integral_constant<int, 0>{}, y_first);
            if (!y_first) sweep(std::integral_constant<int, 1>{}, true);
        }
    });
    return hipGetLastError();
}

hipError_t launch_fluid_speed(const WaveTables &t, const FluidGrid &fg, const double *Q, double *W, double *T,
                              double dx, double dy, unsigned long long *out, hipStream_t s)
{
    const Grid g{t.ns, fg.nx, fg.ny, fg.bc, (long long)fg.nx * fg.ny};
    launch_prim(t, g, Q, W, T, s);
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
