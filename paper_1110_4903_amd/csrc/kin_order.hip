// kin_order.hip -- cost order of an instance's cells for its next advance.
//
// The advance kernels hand cells to lanes (or wavefronts) from a work counter, so a launch
// ends when its last cells finish; cells that need many Newton iterations and are taken late
// leave the rest of the device idle.  The iterations a cell needed in the previous advance of
// the same instance predict its cost well, so the next advance takes the cells in kOrderClasses
// geometric classes, most expensive first: >= 320, 160-319, ..., 10-19, 5-9 and < 5
// iterations.  A first advance (no counts yet) passes classes computed from the source term (direct):
// by the lane kernels' module in that layout, by cost_key_kernel in the others.  Within a class cells
// keep their index order, which keeps the state accesses of neighbouring lanes coalesced.  Which cell a
// lane takes does not change that cell's arithmetic: results are bitwise the same in any order.
//
// A stable counting sort in three kernels over tiles of kOrderTile cells: per-tile class
// counts, one block that turns them into each tile's first position per class, and a scatter
// that ranks a tile's cells within their class by wavefront ballots.  Up to kOrderSmall cells one block
// does it all: there a launch that orders is short enough to feel two launches more.
#include <hip/hip_runtime.h>

#include "kin_internal.h"

namespace kin {
namespace {

#include "kin_xlane.h"

constexpr int kC = kOrderClasses;
constexpr int kOrderThreads = 256;
constexpr int kOrderRounds = kOrderTile / kOrderThreads;
constexpr int kScanThreads = 1024;

// class of a cell that needed `it` iterations: 0 below 5, then one class per doubling; with
// direct, the key is the class
__device__ __forceinline__ int cost_class(int it, int direct)
{
    if (direct) return it < 0 ? 0 : (it >= kC ? kC - 1 : it);
    int k = 0;
#pragma unroll
    for (int b = 5; b <= (5 << (kC - 2)); b <<= 1) k += it >= b;
    return k;
}

// ocount[kC t + c] = cells of class c in tile t
__global__ void __launch_bounds__(kOrderThreads) order_count_kernel(const int *iters, long long n, int direct,
                                                                    int *ocount)
{
    __shared__ int cnt[kC];
    if (threadIdx.x < kC) cnt[threadIdx.x] = 0;
    __syncthreads();
    const long long t0 = (long long)blockIdx.x * kOrderTile;
    for (int r = 0; r < kOrderRounds; ++r) {
        const long long i = t0 + (long long)r * kOrderThreads + threadIdx.x;
        if (i < n) atomicAdd(&cnt[cost_class(iters[i], direct)], 1);
    }
    __syncthreads();
    if (threadIdx.x < kC) ocount[(size_t)blockIdx.x * kC + threadIdx.x] = cnt[threadIdx.x];
}

// In place: ocount[kC t + c] becomes the first position of tile t's class-c cells.  Classes
// are laid out from kC - 1 down to 0; within a class, tiles in order.  One block of T threads; thread u
// owns a contiguous run of tiles.
template <int T>
__global__ void __launch_bounds__(T) order_scan_kernel(int *ocount, long long tiles, unsigned long long *clear)
{
    if (clear && threadIdx.x == 0) *clear = 0ull;  // the advance's work counter
    __shared__ int sc[kC][T];
    __shared__ int tot[kC];
    const int u = threadIdx.x;
    const long long per = (tiles + T - 1) / T;
    const long long b0 = (long long)u * per, b1 = b0 + per < tiles ? b0 + per : tiles;
    int s[kC];
#pragma unroll
    for (int c = 0; c < kC; ++c) s[c] = 0;
    for (long long b = b0; b < b1; ++b)
#pragma unroll
        for (int c = 0; c < kC; ++c) s[c] += ocount[b * kC + c];
#pragma unroll
    for (int c = 0; c < kC; ++c) sc[c][u] = s[c];
    __syncthreads();
    // inclusive scans over the threads (Hillis-Steele)
    for (int d = 1; d < T; d <<= 1) {
        int v[kC];
#pragma unroll
        for (int c = 0; c < kC; ++c) v[c] = u >= d ? sc[c][u - d] : 0;
        __syncthreads();
#pragma unroll
        for (int c = 0; c < kC; ++c) sc[c][u] += v[c];
        __syncthreads();
    }
    if (u < kC) tot[u] = sc[u][T - 1];
    __syncthreads();
    int run[kC];
    int acc = 0;
#pragma unroll
    for (int c = kC - 1; c >= 0; --c) {
        run[c] = acc + sc[c][u] - s[c];
        acc += tot[c];
    }
    for (long long b = b0; b < b1; ++b)
#pragma unroll
        for (int c = 0; c < kC; ++c) {
            const int k = ocount[b * kC + c];
            ocount[b * kC + c] = run[c];
            run[c] += k;
        }
}

// order[position] = cell, stable within each class
__global__ void __launch_bounds__(kOrderThreads) order_scatter_kernel(const int *iters, long long n, int direct,
                                                                      const int *ocount, int *order)
{
    constexpr int kWaves = kOrderThreads / 64;
    __shared__ int run[kC];
    __shared__ int wcnt[kWaves][kC];
    if (threadIdx.x < kC) run[threadIdx.x] = ocount[(size_t)blockIdx.x * kC + threadIdx.x];
    __syncthreads();
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const long long t0 = (long long)blockIdx.x * kOrderTile;
    for (int r = 0; r < kOrderRounds; ++r) {
        const long long i = t0 + (long long)r * kOrderThreads + threadIdx.x;
        const bool valid = i < n;
        const int k = valid ? cost_class(iters[i], direct) : -1;
        unsigned long long mine = 0;
#pragma unroll
        for (int c = 0; c < kC; ++c) {
            const unsigned long long b = __ballot(k == c);
            if (k == c) mine = b;
            if (lane == 0) wcnt[w][c] = __popcll(b);
        }
        __syncthreads();
        if (valid) {
            const int rank = __builtin_amdgcn_mbcnt_hi((unsigned)(mine >> 32),
                                                       __builtin_amdgcn_mbcnt_lo((unsigned)mine, 0u));
            int p = run[k] + rank;
            for (int w2 = 0; w2 < w; ++w2) p += wcnt[w2][k];
            if (p >= 0 && p < n) order[p] = (int)i;
        }
        __syncthreads();
        if (threadIdx.x < kC) {
            int add = 0;
            for (int w2 = 0; w2 < kWaves; ++w2) add += wcnt[w2][threadIdx.x];
            run[threadIdx.x] += add;
        }
        __syncthreads();
    }
}

// The same of at most kOrderSmall cells in one block: a thread counts the classes of its run of cells, 16 bits
// a class, the block scans the counts, and every cell takes its place.  A first advance of inert cells of 36
// species, us in index order, with three kernels and with this one: 2560 cells 199, 224 and 207; 4096 cells
// 294, 316 and 304; 8192 cells 462, 495 and 482 (32768 cells in one block: 1600 with three, 1638 with one;
// one wavefront instead of sixteen: 230, 335 and 553).
constexpr int kSmallRun = 8, kOrderSmall = kSmallRun * kScanThreads;

__global__ void __launch_bounds__(kScanThreads) order_small_kernel(const int *iters, int n, int direct, int *order,
                                                                   unsigned long long *clear)
{
    static_assert(kC == 8 && kOrderSmall < 65536, "two words of four 16-bit counts");
    constexpr int kWaves = kScanThreads / 64;
    __shared__ unsigned long long part[kWaves][2];
    const int u = threadIdx.x, lane = u & 63, w = u >> 6;
    if (clear && u == 0) *clear = 0ull;   // the advance's work counter
    const int per = (n + kScanThreads - 1) / kScanThreads;
    const int a = min(u * per, n), b = min(a + per, n);
    int f[kSmallRun];   // 0..7 are the classes kC - 1..0, in the order of their places
#pragma unroll
    for (int j = 0; j < kSmallRun; ++j) f[j] = a + j < b ? kC - 1 - cost_class(iters[a + j], direct) : 0;
    unsigned long long own[2] = {0, 0}, sum[2];
#pragma unroll
    for (int j = 0; j < kSmallRun; ++j) {
        const unsigned long long one = a + j < b ? 1ull << (16 * (f[j] & 3)) : 0;
        own[0] += f[j] < 4 ? one : 0;
        own[1] += f[j] < 4 ? 0 : one;
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        sum[q] = own[q];
        for (int d = 1; d < 64; d <<= 1) {
            const unsigned long long v = __shfl_up(sum[q], d);
            if (lane >= d) sum[q] += v;
        }
        if (lane == 63) part[w][q] = sum[q];
    }
    __syncthreads();
    unsigned long long all[2] = {0, 0}, next[2] = {sum[0] - own[0], sum[1] - own[1]};
#pragma unroll
    for (int k = 0; k < kWaves; ++k)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const unsigned long long v = part[k][q];
            next[q] += k < w ? v : 0;
            all[q] += v;
        }
    // next: cells of each class in the threads before this one; with the classes before it, the next place
    unsigned long long at = 0;
#pragma unroll
    for (int c = 0; c < kC; ++c) {
        next[c >> 2] += at << (16 * (c & 3));
        at += all[c >> 2] >> (16 * (c & 3)) & 0xffff;
    }
#pragma unroll
    for (int j = 0; j < kSmallRun; ++j)
        if (a + j < b) {
            const int sh = 16 * (f[j] & 3);
            const int p = (int)((f[j] < 4 ? next[0] : next[1]) >> sh & 0xffff);
            if (f[j] < 4) next[0] += 1ull << sh;
            else next[1] += 1ull << sh;
            if (p < n) order[p] = a + j;
        }
}

// Cost class of each cell for a first advance, one wavefront per cell, by the relative temperature change
// that the source term predicts over dt, p = |dT/dt| dt / T: a class takes four octaves of p, from 0 below
// 1 / 16 (and cells that the advance refuses) to 7 above 2^20 (and where p is no number).  The iterations that
// a cell then needs grow by some 35 for four octaves; the rank correlation of p with them is 0.95 to 0.98 (36
// and 100 species, dt = 1e-8 to 1e-6 s), the temperature's own 0.88 to 0.91.  With
// de = sum_r q_r (sum_s nu_sr (h_s - 1)) R T / rho, dT/dt = -de / c_v: one pass over the reactions, without the
// Jacobian.
__global__ void __launch_bounds__(64) cost_key_kernel(WaveTables t, const double *rhos, const double *Ts, const double *Y,
                                                      long long n, long long first, double dt, int *key)
{
    extern __shared__ double sm[];
    const int ns = t.ns, lane = threadIdx.x;
    const long long cell = first + blockIdx.x;
    if (cell >= n) return;
    double *c = sm, *g = sm + ns, *hh = sm + 2 * ns, *Mc = sm + 3 * ns;
    const double rho = rhos[cell], T = Ts[cell];
    bool fin = rho > 0.0 && __builtin_isfinite(rho) && T >= kTmin && T <= kTmax;
    const double iT = 1.0 / T, lT = log(T), rc = 1e-3 * rho, lPaRT = t.lnPaR - lT;
    double cv = 0.0;
    for (int s = lane; s < ns; s += kW) {
        const double y = Y[(size_t)s * n + cell], im = 1.0 / t.M[s];
        fin = fin && __builtin_isfinite(y);
        const double *a = t.nasa + 14 * s + (T < t.Tmid[s] ? 0 : 7);
        const double cp = fma(T, fma(T, fma(T, fma(T, a[4], a[3]), a[2]), a[1]), a[0]);
        const double h = fma(a[5], iT, fma(T, fma(T, fma(T, fma(T, a[4] * 0.2, a[3] * 0.25), a[2] * (1.0 / 3.0)), a[1] * 0.5), a[0]));
        const double e = fma(a[0], lT, fma(T, fma(T, fma(T, fma(T, a[4] * 0.25, a[3] * (1.0 / 3.0)), a[2] * 0.5), a[1]), a[6]));
        c[s] = y * (rc * im);
        g[s] = h - e;
        hh[s] = h;
        cv = fma(y * im, cp - 1.0, cv);
    }
    wave_sync();
    for (int q = lane; q < t.ntb; q += kW) {
        double acc = 0.0;
#pragma unroll 8
        for (int s = 0; s < ns; ++s) acc = fma(t.effT[(size_t)s * t.ntb + q], c[s], acc);
        Mc[q] = acc;
    }
    wave_sync();
    const double4 *rxd4 = reinterpret_cast<const double4 *>(t.rxd);
    double de = 0.0;
    for (int r = lane; r < t.nr; r += kW) {
        const RxnRec x = t.rxc[r];
        const double4 rd = rxd4[r];   // ln A, b, Ta, sum nu
        double p[2] = {1.0, 1.0}, sg = 0.0, sh = 0.0;
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            const int s = x.coff[q] / 8, nu = x.nu[q], m = nu < 0 ? -nu : nu;
            sg = fma((double)nu, g[s], sg);
            sh = fma((double)nu, hh[s], sh);
            for (int k = 0; k < m; ++k) p[q / 3] *= c[s];
        }
        const double lkf = fma(-rd.z, iT, fma(rd.y, lT, rd.x));
        const double pf = exp(lkf) * p[0], pb = x.rev ? exp(lkf - (rd.w * lPaRT - sg)) * p[1] : 0.0;
        de = fma((x.tb >= 0 ? Mc[x.tb] : 1.0) * (pf - pb), sh - rd.w, de);
    }
    const double P = fabs(wave_sum(de)) * dt / (rc * wave_sum(cv));   // |dT/dt| dt / T: R T cancels
    const bool ok = __all(fin);
    int k = 0;
    if (ok) {
        if (!(P < 1e9)) k = kC - 1;
        else if (P > 0.0) k = min(max((int)floor(0.25 * log2(P)) + 2, 0), kC - 1);
    }
    if (lane == 0) key[cell] = k;
}

}  // namespace

hipError_t launch_cost_key(const WaveTables &t, const Arena &a, long long n, double dt, int *key, hipStream_t s)
{
    const size_t lds = sizeof(double) * (size_t)(3 * t.ns + t.ntb);
    // a grid holds less than 2^32 threads, so the cells go in parts of half as many
    constexpr long long kPart = (1ll << 31) / kW;
    for (long long first = 0; first < n; first += kPart) {
        const long long m = n - first < kPart ? n - first : kPart;
        hipLaunchKernelGGL(cost_key_kernel, dim3((unsigned)m), dim3(kW), lds, s, t, a.rho, a.T, a.Y, n, first, dt, key);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_cost_order(const int *key, long long n, bool direct, int *order, int *ocount,
                              unsigned long long *clear, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    if (n > 0x7fffffffLL) return hipErrorInvalidValue;
    const long long tiles = order_tiles(n);
    const int d = direct ? 1 : 0;
    if (n <= kOrderSmall) {
        hipLaunchKernelGGL(order_small_kernel, dim3(1), dim3(kScanThreads), 0, s, key, (int)n, d, order, clear);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(order_count_kernel, dim3((unsigned)tiles), dim3(kOrderThreads), 0, s, key, n, d, ocount);
    // One wavefront where a lane has a tile at most: on a device that other streams keep full it starts as
    // soon as any wavefront of theirs ends, a block of sixteen when a compute unit has run empty (serving 160
    // requests, mean time in the queue and running: 0.05 to 0.1 ms, and 3 ms).
    if (tiles <= 64) hipLaunchKernelGGL(order_scan_kernel<64>, dim3(1), dim3(64), 0, s, ocount, tiles, clear);
    else hipLaunchKernelGGL(order_scan_kernel<kScanThreads>, dim3(1), dim3(kScanThreads), 0, s, ocount, tiles, clear);
    hipLaunchKernelGGL(order_scatter_kernel, dim3((unsigned)tiles), dim3(kOrderThreads), 0, s, key, n, d, ocount,
                       order);
    return hipGetLastError();
}

}  // namespace kin
