// The gfx950 MFM hydro pass: kernel length, flux lists, gradients, fluxes.
//
// One thread, or a few that share its list, per (Morton-ordered) particle; blocks are remapped so that each
// XCD works on one contiguous run of particles and keeps its neighbours in
// its own L2.  The flux kernel evaluates every unordered pair on both of its
// particles with the lower index as the left state, so both copies are
// bitwise equal and the accumulated momentum and energy cancel exactly pair
// by pair; there are no atomics on outputs and results are deterministic.
#include <algorithm>
#include <limits.h>
#include <math.h>

#include <type_traits>

#include "device.h"
#include "kernels.h"

namespace mfm {

// blockIdx -> logical block so that XCD x (blocks x, x+8, ...) gets one contiguous range
__device__ __forceinline__ int xcd_block() {
    int G = gridDim.x, b = blockIdx.x;
    int x = b & 7, slot = b >> 3;
    int q = G >> 3, r = G & 7;
    return x * q + (x < r ? x : r) + slot;
}

__device__ __forceinline__ void count_add(unsigned long long* c, unsigned long long v) {
    v = wave_reduce(v, [](unsigned long long a, unsigned long long b) { return a + b; });
    if ((threadIdx.x & 63) == 0 && v) atomicAdd(c, v);
}

// the atomic is skipped when the counter already holds at least v (a stale
// read only costs an atomic that changes nothing)
__device__ __forceinline__ void count_max(unsigned long long* c, unsigned long long v) {
    v = wave_reduce(v, [](unsigned long long a, unsigned long long b) { return a > b ? a : b; });
    if ((threadIdx.x & 63) == 0 && v && v > __atomic_load_n(c, __ATOMIC_RELAXED)) atomicMax(c, v);
}

__device__ __forceinline__ void flag_index(Counters* cnt, int i) {
    atomicMin(&cnt->first_bad, (unsigned long long)i);
}

__device__ __forceinline__ void displacement(const Phys& ph, const double xi[3], double xj0, double xj1,
                                             double xj2, double d[3]) {
    d[0] = min_image(xj0 - xi[0], ph.box[0], ph.periodic[0]);
    d[1] = min_image(xj1 - xi[1], ph.box[1], ph.periodic[1]);
    d[2] = min_image(xj2 - xi[2], ph.box[2], ph.periodic[2]);
}

// ------------------------------------------------------------ kernel length
// The root of (32/3) sum_j w(r_ij / H) = n_ngb is found per particle by
// safeguarded Newton iterations on the radii r_ij < hi of a bracket (lo, hi].
// A scan at a trial radius R collects the radii (rl) and indices (jl) within R
// into interleaved global lists (rl[k * n + i], coalesced across a wave); a
// lane whose R holds too few neighbours, or more than the list holds, adjusts R
// and scans again.  Scans are wave-cooperative: each pass takes the lanes whose
// trial radius is within a factor two of the largest one and lie close to the
// first of them, and scans their union once.  Particles the first round leaves
// without a bracket go to the per-particle list solver, one wave each, and the
// few it cannot finish to the rescanning solver.  After the root, the indices
// with r < H (self excluded) are compacted in place: the gather part of the
// flux list.

// Local density from the 3x3x3 blocks of cells around the particle's own cell:
// on the finest level l whose block holds at least kColdCount particles, and on
// level l + 1, whose block holds fewer.  log(count) is interpolated linearly in
// log(volume) between the two blocks to the volume that holds kColdCount
// particles; the guess is the radius holding n_ngb particles at that density.
// The interpolation removes most of the factor-of-8 steps between levels (on
// the clustered log-normal set the spread of log(H / guess) drops from 0.22 to
// 0.18 and the particles left without a bracket by the first scan from 17% to
// 11%).  A smaller kColdCount gives a more local estimate but a noisier one
// from particle to particle, which widens the cooperative scans (they reach the
// largest trial radius of the lanes they serve) by more than it saves.  Open
// sides shrink the blocks to the cells inside.  The search starts at the level
// where a block at the mean density would hold kColdCount particles and moves
// finer or coarser from there.
constexpr double kColdCount = 32.0;
struct BlockCount {
    double count;
    double vol;
};

// the level-l block around the cell of a particle with the (full-depth) key;
// the level is the same on every lane
__device__ BlockCount block_count(const TreeDesc& td, const int2* __restrict__ tab, unsigned long long key, int l) {
    unsigned long long dil[3][3];   // key bits of coordinates c-1, c, c+1 per axis
    bool ok[3][3];
    int ncl[3];
    const unsigned long long cell = key >> (td.ktot - td.kbits[l]);
#pragma unroll
    for (int d = 0; d < 3; d++) {
        const int nc = td.ncell[l][d];
        // the neighbours c - 1 and c + 1 by dilated subtraction and addition of
        // the lowest key bit of the axis (wrapping modulo nc, which only periodic
        // axes use); c is 0 or nc - 1 where none or all of the axis's bits are set
        const unsigned long long m = td.mask[l][d];
        const unsigned long long one = m & (~m + 1);
        const unsigned long long dc = cell & m;
        dil[d][0] = dilated_sub(dc, one, m);
        dil[d][1] = dc;
        dil[d][2] = dilated_add(dc, one, m);
        // fewer than 3 cells: count each once
        ok[d][0] = nc >= 3 && (td.periodic[d] || dc != 0);
        ok[d][1] = true;
        ok[d][2] = nc >= 3 && (td.periodic[d] || dc != m);
        ncl[d] = 1 + ok[d][0] + ok[d][2];
    }
    int cnt = 0;
    const int2* __restrict__ cells = tab + td.tab_off[l];
#pragma unroll
    for (int ox = 0; ox < 3; ox++)
#pragma unroll
        for (int oy = 0; oy < 3; oy++)
#pragma unroll
            for (int oz = 0; oz < 3; oz++) {
                // cells outside an open side read cell 0 and count nothing
                const bool in = ok[0][ox] && ok[1][oy] && ok[2][oz];
                const int2 se = cells[in ? (dil[0][ox] | dil[1][oy] | dil[2][oz]) : 0ull];
                cnt += in ? se.y - se.x : 0;
            }
    return {(double)cnt, ncl[0] * td.cs[l][0] * ncl[1] * td.cs[l][1] * ncl[2] * td.cs[l][2]};
}

// every lane of the wave takes part; the lanes with `want` get a guess
__device__ double cold_guess(const TreeDesc& td, const int2* __restrict__ tab, unsigned long long key, bool want,
                             double n_ngb, long long n) {
    const double need = kColdCount;
    const double nbox = (double)n / (td.box[0] * td.box[1] * td.box[2]);
    int l0 = td.bmax;
    while (l0 > 0 && 27.0 * nbox * td.cs[l0][0] * td.cs[l0][1] * td.cs[l0][2] < need) l0--;
    l0 = __builtin_amdgcn_readfirstlane(l0);
    BlockCount b = {0.0, 0.0};
    BlockCount f = {-1.0, 0.0};   // the finer block (count < need), once known
    if (want) b = block_count(td, tab, key, l0);
    bool finer = want && b.count >= need, coarser = want && !finer;
    for (int l = l0 + 1; l <= td.bmax && __ballot(finer); l++)
        if (finer) {
            const BlockCount g = block_count(td, tab, key, l);
            if (g.count < need) {
                f = g;
                finer = false;
            } else {
                b = g;
            }
        }
    for (int l = l0 - 1; l >= 0 && __ballot(coarser); l--)
        if (coarser) {
            f = b;
            b = block_count(td, tab, key, l);
            coarser = b.count < need;
        }
    double vol = b.vol, count = fmax(b.count, 1.0);
    if (f.count >= 0.0 && b.count >= need && f.vol < b.vol) {
        // log count linear in log volume between the two blocks, at count = need
        const double lf = log(fmax(f.count, 0.5)), lb = log(b.count);
        const double t = (log(need) - lf) / (lb - lf);
        vol = exp(log(f.vol) + t * (log(b.vol) - log(f.vol)));
        count = need;
    }
    return cbrt(3.0 * n_ngb * vol / (4.0 * M_PI * count));
}

// products and sums rounded one by one (contraction into fma is switched off
// here), so that an expression gives the same bits wherever it is compiled: the
// face sum whichever owner evaluates it, a residual whichever kernel forms it
template <typename T>
__device__ __forceinline__ T mul_rn(T x, T y) {
#pragma clang fp contract(off)
    return x * y;
}
template <typename T>
__device__ __forceinline__ T add_rn(T x, T y) {
#pragma clang fp contract(off)
    return x + y;
}

constexpr double kNewtonTail = 1e-9;   // last Newton step accepted without a check pass

// One safeguarded Newton update from the residual f and slope fp at Hc, inside
// the bracket (lo, hi]; true when Hc is final.  The sum is twice continuously
// differentiable in H (so is the spline), so Newton converges quadratically:
// after a step below kNewtonTail H the new iterate is within a small multiple
// of kNewtonTail^2 H (a few 1e-18 relative) of the root and is returned without
// another pass.  It is taken even at a bracket edge: an earlier iterate can
// land on the root and become lo or hi.
__device__ __forceinline__ bool newton_step(double f, double fp, double& lo, double& hi, double& Hc) {
    if (f == 0.0) return true;
    if (f < 0.0) lo = Hc;
    else hi = Hc;
    double Hn = Hc - f / fp;
    if (fabs(Hn - Hc) <= kNewtonTail * Hc) {
        Hc = fmin(hi, fmax(lo, Hn));
        return true;
    }
    if (!(Hn > lo && Hn <= hi)) Hn = 0.5 * (lo + hi);
    const double dH = fabs(Hn - Hc);
    Hc = Hn;
    return dH <= 1e-14 * Hc || !(hi - lo > 4e-16 * hi);
}

// Each particle takes one group scan; those it does not finish (no bracket, or
// more radii than the list holds) go to the per-particle solver, which is
// cheaper for them than further group passes over a sparse class.
constexpr double kColdPad = 1.05;   // scan radius over a cold guess
constexpr double kWarmPad = 1.03;   // scan radius over the previous H
// Four waves per SIMD: 128 VGPRs, and the 37 KB of staged candidates per block
// fit four times in the LDS of a compute unit.
// With HIER (hierarchical steps with active subsets) only the particles of
// mode 1 solve; the others keep their kernel length.  The cell tables may then
// be those of an earlier build: every scan reaches *pad further, the largest
// distance a particle has moved since.
constexpr int kSolveWaves = 4;
template <bool HIER>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kSolveWaves))) void k_solve_h(PassArrays a, TreeDesc td, const int2* __restrict__ tab,
                                                  const double4* __restrict__ pos, const unsigned long long* __restrict__ keys, Phys ph,
                                                  Counters* cnt, double* __restrict__ rl, int* __restrict__ jl,
                                                  int* __restrict__ gcount, int* __restrict__ counts,
                                                  int* __restrict__ fb_list, unsigned long long* __restrict__ fb_count,
                                                  const unsigned char* __restrict__ mode, const double* __restrict__ pad) {
    cnt = counter_copy(cnt);
    __shared__ GroupLds lds[256 / kWave];
    GroupLds& S = lds[threadIdx.x / kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int i = xcd_block() * 256 + threadIdx.x;
    const bool act = i < a.n && (!HIER || mode[i] == kModeSolve);
    const long long n = a.n;
    const int cap = min(kRCap, ph.max_ngb);
    const double c32 = 32.0 / 3.0;
    double half = INFINITY;
    for (int d = 0; d < 3; d++)
        if (ph.periodic[d]) half = fmin(half, 0.5 * ph.box[d]);
    double xi[3] = {0.0, 0.0, 0.0};
    double R = 0.0, guess = 0.0;   // scan radius
    bool warm = false;
    if (act) {
        const double4 pi = pos[i];
        xi[0] = pi.x;
        xi[1] = pi.y;
        xi[2] = pi.z;
        guess = a.H[i];
        warm = guess > 0.0;
    }
    if (__ballot(act && !warm)) {
        const double g = cold_guess(td, tab, act ? keys[i] : 0ull, act && !warm, ph.n_ngb, a.n);
        if (!warm) guess = g;
    }
    if (act) {
        R = (warm ? kWarmPad : kColdPad) * guess;
        if (R >= half) R = half * (1.0 - 1e-12);
    }
    // Weighted counts at R and at two trial lengths: below the guess (at it on a
    // cold start) and at the scan radius again, formed from the guess.
    const double Hg = R * (warm ? 1.0 / kWarmPad : 1.0 / kColdPad);
    const double Ht0 = warm ? 0.97 * Hg : Hg, Ht1 = (warm ? kWarmPad : kColdPad) * Hg;
    double sw = 0.0, st0 = 0.0, st1 = 0.0;
    int m = 0;   // radii met, listed while they fit
    double* __restrict__ rp = rl + i;
    int* __restrict__ jp = jl + i;
    bool need = act && R > 0.0;
    // A group whose scan spans a periodic axis whole (a thin box) is left to the list
    // solver, whose single spheres rarely do: its tests would need the minimum image
    // of every pair, off the matrix cores.  Measured (solve stage, shock tubes of
    // 14, 18 and 24 spacings across): 549 -> 238, 653 -> 200, 840 -> 273 us.
    bool unmade = false;
    for (int pass = 0; pass < kWave; pass++) {
        if (__ballot(need) == 0) break;
        const ScanClass cl = scan_class(need, R, xi);
        const double iR = 1.0 / R, iT0 = 1.0 / Ht0, iT1 = 1.0 / Ht1;
        const bool made = group_scan<false>(td, tab, pos, S, lane, cl.bmin, cl.bmax, cl.Rq, HIER ? *pad : 0.0, xi, R * R, cl.in, [&](int j, double r2) {
            const double r = sqrt_mid(r2);
            if (m < cap) {
                *rp = r;
                *jp = j;
            }
            rp += n;
            jp += n;
            m++;
            sw += spline_w(r * iR);
            st0 += spline_w(r * iT0);
            st1 += spline_w(r * iT1);
        });
        unmade = unmade || (cl.in && !made);
        need = need && !cl.in;
    }
    // A bracket with every radius below it listed is narrowed by the trial counts
    // (summed in the order of the Newton sums, so the signs agree).  Newton starts
    // from the secant of the bracket when both ends carry a residual, else from
    // the density scaling of the upper end.
    const double neff = c32 * sw;
    double lo = 0.0, hi = R, neff_hi = neff, fa = NAN;
    const bool found = act && neff >= ph.n_ngb && m <= cap;
    if (found) {
        const double f0 = add_rn(mul_rn(c32, st0), -ph.n_ngb), f1 = add_rn(mul_rn(c32, st1), -ph.n_ngb);
        if (Ht1 < hi) {
            if (f1 >= 0.0) hi = Ht1, neff_hi = f1 + ph.n_ngb;
            else lo = Ht1, fa = f1;
        }
        if (Ht0 < hi && Ht0 > lo) {
            if (f0 >= 0.0) hi = Ht0, neff_hi = f0 + ph.n_ngb;
            else lo = Ht0, fa = f0;
        }
    }
    if (found) {
        // Newton's start and bracket, for the root kernel
        const double fb = neff_hi - ph.n_ngb;
        double Hc;
        if (fa < 0.0 && fb >= 0.0) Hc = lo + (hi - lo) * (-fa / (fb - fa));
        else Hc = (warm && guess > lo && guess < hi) ? guess : hi * cbrt(ph.n_ngb / neff_hi);
        if (!(Hc > lo && Hc <= hi)) Hc = 0.5 * (lo + hi);
        a.H[i] = Hc;
        a.nk[i] = lo;
        a.V[i] = hi;
        gcount[i] = m;
    } else if (act) {
        // hand over to the per-particle solver: the bracket and the next trial
        // radius, in the particle's own (now unused) radius slots 0-2
        double Rn = R;
        if (!(R > 0.0) || unmade) {
            // no scan without a radius (positions that are not numbers), or none made
            hi = INFINITY;
        } else if (!(neff >= ph.n_ngb)) {
            // grow by the density estimate, at least 1.15x, at most 4x
            lo = R;
            hi = INFINITY;
            Rn = R * fmin(4.0, fmax(1.15, 1.1 * cbrt(ph.n_ngb / fmax(neff, 1e-300))));
        } else if (m > cap) {
            // bracketed, but too many radii to keep: just above the estimated root
            Rn = fmax(lo + 0.25 * (hi - lo), fmin(1.05 * R * cbrt(ph.n_ngb / neff), R * cbrt(0.8 * cap / m)));
            if (!(Rn < hi)) Rn = 0.5 * (lo + hi);
        }
        const unsigned long long slot = atomicAdd(fb_count, 1ull);
        if (slot < (unsigned long long)a.n) fb_list[slot] = i;
        rl[i] = lo;
        rl[n + i] = hi;
        rl[2 * n + i] = Rn;
        a.H[i] = hi < INFINITY ? hi : (lo > 0.0 ? lo : guess);
        gcount[i] = 0;   // nothing for the root kernel
    }
    count_add(&cnt->h_iters, act ? 1ull : 0ull);
    count_max(&cnt->h_iters_max, act ? 1ull : 0ull);
    count_max(&cnt->h_rounds_max, act ? 1ull : 0ull);
}

// The root of each particle the group scan bracketed, one thread per particle:
// safeguarded Newton on its listed radii from the start in H and the bracket
// in nk and V, then nk, V and the gather list.  The first kRootRadii radii sit
// in registers (every index fixed at compile time, a wave runs as far as its
// longest list; slots past a lane's own hold a radius beyond the bracket, whose
// terms are zero), so the list is read once: read again by every iteration at
// the scan kernel's four waves per SIMD, this part waited on the lists for
// 0.53 of the scan's 1.34 ms (lattice, 2.1M) and 11 of 29 ms (clustered, 16.8M).
// Three waves per SIMD hold 64 radii each, which covers most waves' lists.
// Measured (solve stage): lattice 2.1M 1.41 -> 1.29 ms, clustered 16.8M
// 36.8 -> 31.7 ms.
constexpr int kRootRadii = 64;
constexpr int kRootBlock = 8;
constexpr int kRootWaves = 3;
template <bool HIER>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kRootWaves))) void k_root_h(
    PassArrays a, double n_ngb, int maxit, Counters* cnt, double* __restrict__ rl, int* __restrict__ jl,
    int* __restrict__ gcount, int* __restrict__ counts, int* __restrict__ fb_list,
    unsigned long long* __restrict__ fb_count, const unsigned char* __restrict__ mode) {
    cnt = counter_copy(cnt);
    const int i = xcd_block() * 256 + threadIdx.x;
    const long long n = a.n;
    const double c32 = 32.0 / 3.0;
    int m = 0;
    double Hc = 1.0, lo = 0.0, hi = 1.0;
    if (i < a.n && (!HIER || mode[i] == kModeSolve)) m = gcount[i];
    if (m > 0) {
        Hc = a.H[i];
        lo = a.nk[i];
        hi = a.V[i];
    }
    const int kmax = __builtin_amdgcn_readfirstlane(wave_max_i(min(m, kRootRadii)));
    double r[kRootRadii];
#pragma unroll
    for (int b = 0; b < kRootRadii; b += kRootBlock)
        if (b < kmax) {
#pragma unroll
            for (int k = b; k < b + kRootBlock; k++) r[k] = k < m ? rl[k * n + i] : 2.0 * hi;
        }
    unsigned long long iters = 0;
    bool conv = false;
    if (m > 0) {
        for (int it = 0; it < maxit; it++) {
            iters++;
            const double iH = 1.0 / Hc;
            double s = 0.0, sq = 0.0;
#pragma unroll
            for (int b = 0; b < kRootRadii; b += kRootBlock)
                if (b < kmax) {
#pragma unroll
                    for (int k = b; k < b + kRootBlock; k++) {
                        const double q = r[k] * iH;
                        s += spline_w(q);
                        sq += spline_qdw(q);
                    }
                }
#pragma unroll 4
            for (int k = kRootRadii; k < m; k++) {
                const double q = rl[k * n + i] * iH;
                s += spline_w(q);
                sq += spline_qdw(q);
            }
            if (newton_step(add_rn(mul_rn(c32, s), -n_ngb), -c32 * sq * iH, lo, hi, Hc)) {
                conv = true;
                break;
            }
        }
    }
    if (conv) {
        // the indices with r < H but the particle itself, compacted in place (a
        // block's indices are read before any slot of the block is written)
        double sum = 0.0;
        const double iH = 1.0 / Hc;
        int c = 0;
#pragma unroll
        for (int b = 0; b < kRootRadii; b += kRootBlock)
            if (b < kmax) {
                int j[kRootBlock];
#pragma unroll
                for (int k = 0; k < kRootBlock; k++) j[k] = b + k < m ? jl[(b + k) * n + i] : i;
#pragma unroll
                for (int k = 0; k < kRootBlock; k++) {
                    sum += spline_w(r[b + k] * iH);
                    if (r[b + k] < Hc && j[k] != i) {
                        jl[c * n + i] = j[k];
                        c++;
                    }
                }
            }
        for (int k = kRootRadii; k < m; k++) {
            const double rk = rl[k * n + i];
            sum += spline_w(rk * iH);
            const int j = jl[k * n + i];
            if (rk < Hc && j != i) {
                jl[c * n + i] = j;
                c++;
            }
        }
        const double nk = kernel_norm(Hc) * sum;
        a.H[i] = Hc;
        a.nk[i] = nk;
        a.V[i] = 1.0 / nk;
        gcount[i] = c;
        counts[i] = 0;   // tail entries, appended by the gradient kernel
    } else if (m > 0) {
        // not converged: the bracket goes on to the per-particle solver
        const unsigned long long slot = atomicAdd(fb_count, 1ull);
        if (slot < (unsigned long long)a.n) fb_list[slot] = i;
        rl[i] = lo;
        rl[n + i] = hi;
        rl[2 * n + i] = hi;
        a.H[i] = hi;
    }
    count_add(&cnt->h_iters, iters);
    count_max(&cnt->h_iters_max, iters + 1);
}


// Small sets skip the group scan: every particle starts with its guess as the
// first trial radius and goes to the list solver, one wave each.  Up to
// kDirectMax particles the group scan has too few waves to fill the chip (one
// per 64 particles, for 1,024 SIMDs), and the time is that of one wave's serial
// work: on clustered sets pass after pass over the wave's mixed radii.
// Measured (solve stage, group scan against this way, cold): lattice 4,096
// 89 / 37 us, 13,824 186 / 68, 32,768 89 / 115 (cells and waves aligned), 46,656
// 172 / 161, 64,000 176 / 198; random 46,656 230 / 153, 64,000 253 / 198;
// clustered 4,096 1,098 / 96, 32,768 764 / 205, 64,000 909 / 446.  The line is
// where an even set's time is the same both ways.
constexpr int kDirectMax = 49152;
template <bool HIER>
__global__ __launch_bounds__(256) void k_solve_start(PassArrays a, TreeDesc td, const int2* __restrict__ tab,
                                                     const unsigned long long* __restrict__ keys, Phys ph,
                                                     double* __restrict__ hand, int* __restrict__ fb_list,
                                                     unsigned long long* __restrict__ fb_count,
                                                     unsigned long long* __restrict__ fb2_count,
                                                     const unsigned char* __restrict__ mode) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    const bool act = i < a.n && (!HIER || mode[i] == kModeSolve);
    const long long n = a.n;
    const double H0 = act ? a.H[i] : 0.0;
    const bool warm = H0 > 0.0;
    double guess = H0;
    if (__ballot(act && !warm)) {
        const double g = cold_guess(td, tab, act ? keys[i] : 0ull, act && !warm, ph.n_ngb, a.n);
        if (!warm) guess = g;
    }
    int slot = i;
    if (HIER) {
        const unsigned long long m = __ballot(act);
        unsigned long long base = 0;
        if (m && (threadIdx.x & (kWave - 1)) == 0) base = atomicAdd(fb_count, (unsigned long long)__popcll(m));
        slot = __shfl((int)base, 0, kWave) + __popcll(m & ((1ull << (threadIdx.x & (kWave - 1))) - 1ull));
    } else if (i == 0) {
        *fb_count = (unsigned long long)n;
        *fb2_count = 0ull;
    }
    if (!act) return;
    fb_list[slot] = i;
    hand[i] = 0.0;
    hand[n + i] = INFINITY;
    hand[2 * n + i] = (warm ? kWarmPad : kColdPad) * guess;
}

// Particles the group scan hands over (and all of a small set), one wave each.
// The wave scans the cells within a trial radius once and keeps every radius and index within it in
// registers (entry e on lane e mod 64, slot e / 64, scan order), narrows the
// bracket with the weighted count at that radius, and once the radius brackets
// the root with every radius kept, runs Newton on them with wave-wide sums in
// a fixed order.  Particles whose radii do not fit, or that find no bracket
// within kWaveScans scans, go on to the rescanning solver below.
constexpr int kWaveSlots = 3;   // entries per lane kept by the list solver (ra, rb, rc)
constexpr int kWaveScans = 16;
// At five waves per SIMD 5,120 waves are resident; 32,768 single-wave blocks
// (about 87 particles each on the clustered set) balance the end of the
// launch better than 16,384 (45.2 -> 44.5 ms for the solve stage).
constexpr int kWaveBlocks = 32768;   // waves of the list solver at most, striding over its particles
// a single sphere's scan enumerates its cells at a coarser level than a group's
constexpr double kWaveScanScale = 0.5;

// Five waves per SIMD: the list solver fits in 96 registers without spills,
// and the fifth wave hides more of its scans' load latency than four.
constexpr int kWaveSolveWaves = 5;
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kWaveSolveWaves))) void k_solve_h_wave(
                                                      PassArrays a, TreeDesc td, const int2* __restrict__ tab,
                                                      const double4* __restrict__ pos, Phys ph, Counters* cnt,
                                                      const int* __restrict__ fb_list,
                                                      const unsigned long long* __restrict__ fb_count,
                                                      const double* __restrict__ hand, int* __restrict__ jl,
                                                      int* __restrict__ gcount, int* __restrict__ counts,
                                                      int* __restrict__ fb2_list,
                                                      unsigned long long* __restrict__ fb2_count,
                                                      const double* __restrict__ pad, int scanned) {
    cnt = counter_copy(cnt);
    __shared__ ScanLds S;
    const int lane = threadIdx.x;
    const unsigned long long nfb = min(*fb_count, (unsigned long long)a.n);
    const double pd = pad ? *pad : 0.0;
    if (blockIdx.x == 0 && lane == 0) cnt->h_fallback = *fb_count;
    const long long n = a.n;
    constexpr int kKeep = kWaveSlots * kWave;
    const double c32 = 32.0 / 3.0;
    double half = INFINITY;
    for (int d = 0; d < 3; d++)
        if (ph.periodic[d]) half = fmin(half, 0.5 * ph.box[d]);
    const unsigned long long below = (1ull << lane) - 1ull;
    unsigned long long iters = 0, iters_max = 0, over = 0, scans_max = 0, many = 0;
    for (unsigned long long t = blockIdx.x; t < nfb; t += gridDim.x) {
        const unsigned long long iters0 = iters;
        const int i = __builtin_amdgcn_readfirstlane(fb_list[t]);
        const double4 pi = pos[i];
        const double xi[3] = {uniform_d(pi.x), uniform_d(pi.y), uniform_d(pi.z)};
        double lo = uniform_d(hand[i]), hi = uniform_d(hand[n + i]), R = uniform_d(hand[2 * n + i]);
        if (!(R > lo)) R = (hi < INFINITY) ? hi : 1.3 * lo;
        // the kept entries of this lane: slots 0-2 (named, so they stay in registers)
        double ra = INFINITY, rb = INFINITY, rc = INFINITY;
        int ja = -1, jb = -1, jc = -1;
        int m = 0, scans = 0;
        double neff_hi = 0.0;
        bool bracketed = false;
        while (scans < kWaveScans) {
            if (!(R < half)) R = half * (1.0 - 1e-12);
            if (!(R > lo)) break;
            scans++;
            iters++;
            const double R2 = R * R, iR = 1.0 / R;
            double sw = 0.0;
            m = 0;
            ra = rb = rc = INFINITY;
            ja = jb = jc = -1;
            scan_cells(td, tab, pos, S, lane, xi, xi, R + pd, [&](const double4& q, bool valid, int, int wrap) {
                const double r2 = sq_disp(q, xi, wrap, td.box);
                const bool in = valid && r2 < R2;
                const double r = sqrt(r2);
                if (in) sw += spline_w(r * iR);
                // new entries m .. m + cin - 1 go to lanes (m + rank) mod 64; the
                // other lanes send to the remaining lanes, so every lane gets one value
                const unsigned long long b = __ballot(in);
                const int cin = __popcll(b);
                const int rank = in ? __popcll(b & below) : cin + __popcll(~b & below);
                const int dest = (m + rank) & (kWave - 1);
                const long long rbits = __double_as_longlong(r);
                const int rlo = __builtin_amdgcn_ds_permute(dest * 4, (int)rbits);
                const int rhi = __builtin_amdgcn_ds_permute(dest * 4, (int)(rbits >> 32));
                const int jv = __builtin_amdgcn_ds_permute(dest * 4, (int)__double_as_longlong(q.w));
                const int off = (lane - m) & (kWave - 1);
                if (off < cin) {
                    const int sl = (m + off) / kWave;
                    const double rv = __longlong_as_double(((long long)rhi << 32) | (unsigned)rlo);
                    ra = sl == 0 ? rv : ra;
                    ja = sl == 0 ? jv : ja;
                    rb = sl == 1 ? rv : rb;
                    jb = sl == 1 ? jv : jb;
                    rc = sl == 2 ? rv : rc;
                    jc = sl == 2 ? jv : jc;
                }
                m += cin;
            }, kWaveScanScale);
            sw = uniform_d(wave_sum_d(sw));
            const double neff = c32 * sw;
            if (m > kKeep) {
                // too many radii to keep; below n_ngb the root lies beyond them all
                if (neff < ph.n_ngb) break;
                hi = fmin(hi, R);
                R = fmax(lo + 0.25 * (hi - lo), fmin(1.05 * R * cbrt(ph.n_ngb / neff), R * cbrt(0.8 * kKeep / m)));
                if (!(R < hi)) R = 0.5 * (lo + hi);
            } else if (neff < ph.n_ngb) {
                lo = R;
                if (hi < INFINITY) {
                    R = hi;
                } else {
                    const double g = 1.1 * cbrt(ph.n_ngb / fmax(neff, 1e-300));
                    R *= fmin(4.0, fmax(1.15, g));
                }
            } else {
                hi = R;
                neff_hi = neff;
                bracketed = true;
                break;
            }
        }
        bool conv = false;
        double Hc = hi;
        if (bracketed) {
            Hc = hi * cbrt(ph.n_ngb / neff_hi);
            if (!(Hc > lo && Hc <= hi)) Hc = 0.5 * (lo + hi);
            for (int it = 0; it < ph.h_maxit; it++) {
                iters++;
                const double iH = 1.0 / Hc;
                double s = 0.0, sq = 0.0;
                const double rs[kWaveSlots] = {ra, rb, rc};
#pragma unroll
                for (int sl = 0; sl < kWaveSlots; sl++)
                    if (sl * kWave + lane < m) {
                        const double q = rs[sl] * iH;
                        s += spline_w(q);
                        sq += spline_qdw(q);
                    }
                wave_sum2_d(s, sq, s, sq);
                if (newton_step(c32 * s - ph.n_ngb, -c32 * sq * iH, lo, hi, Hc)) {
                    conv = true;
                    break;
                }
            }
        }
        if (!conv) {
            // on to the rescanning solver, which grows a bracket from a.H
            if (lane == 0) {
                const unsigned long long slot = atomicAdd(fb2_count, 1ull);
                if (slot < (unsigned long long)a.n) fb2_list[slot] = i;
                a.H[i] = (hi < INFINITY) ? hi : R;
            }
            continue;
        }
        // gather list: every kept index with r < H but the particle itself, in scan order
        const double iH = 1.0 / Hc;
        double sum = 0.0;
        int c = 0;
        const double rs[kWaveSlots] = {ra, rb, rc};
        const int js[kWaveSlots] = {ja, jb, jc};
#pragma unroll
        for (int sl = 0; sl < kWaveSlots; sl++) {
            const bool have = sl * kWave + lane < m;
            if (have) sum += spline_w(rs[sl] * iH);
            const bool in = have && rs[sl] < Hc && js[sl] != i;
            const unsigned long long b = __ballot(in);
            const int slot = c + __popcll(b & below);
            if (in && slot < ph.max_ngb) jl[(long long)slot * n + i] = js[sl];
            c += __popcll(b);
        }
        sum = wave_sum_d(sum);
        if (c > ph.max_ngb) {
            c = ph.max_ngb;
            over = 1;
            if (lane == 0) flag_index(cnt, i);
        }
        if (lane == 0) {
            const double nk = kernel_norm(Hc) * sum;
            a.H[i] = Hc;
            a.nk[i] = nk;
            a.V[i] = 1.0 / nk;
            gcount[i] = c;
            counts[i] = 0;
        }
        iters_max = max(iters_max, iters - iters0);
        scans_max = max(scans_max, (unsigned long long)scans);
        many += (scanned + scans >= 3) ? 1ull : 0ull;
    }
    if (lane == 0) {
        if (iters) atomicAdd(&cnt->h_iters, iters);
        if (iters_max) atomicMax(&cnt->h_iters_max, iters_max);
        if (scans_max) atomicMax(&cnt->h_rounds_max, scanned + scans_max);
        if (many) atomicAdd(&cnt->h_rounds3, many);
        if (over) atomicAdd(&cnt->overflow, over);
    }
}

// Solve for the few particles the list solver handed on (no bracket within its
// scans, or more radii than it keeps): one wave per particle,
// every residual evaluation scans the cells within H again with the lanes
// splitting the particles, so there is no limit on the number of neighbours.
// The bracket grows from the handed-over H until it holds the root, then
// Newton with bisection safeguard; a last scan writes the gather list.
__global__ __launch_bounds__(64) void k_solve_h_fallback(PassArrays a, TreeDesc td, const int2* __restrict__ tab,
                                                          const double4* __restrict__ pos, Phys ph, Counters* cnt,
                                                          const int* __restrict__ fb_list,
                                                          const unsigned long long* __restrict__ fb_count,
                                                          int* __restrict__ jl, int* __restrict__ gcount,
                                                          int* __restrict__ counts, const double* __restrict__ pad) {
    cnt = counter_copy(cnt);
    __shared__ ScanLds S;
    const int lane = threadIdx.x;
    const double pd = pad ? *pad : 0.0;
    const unsigned long long nfb = min(*fb_count, (unsigned long long)a.n);
    if (blockIdx.x == 0 && lane == 0) cnt->h_rescan = *fb_count;
    const long long n = a.n;
    const double c32 = 32.0 / 3.0;
    double half = INFINITY;
    for (int d = 0; d < 3; d++)
        if (ph.periodic[d]) half = fmin(half, 0.5 * ph.box[d]);
    unsigned long long iters = 0, iters_max = 0, noconv = 0, noimg = 0, over = 0;
    for (unsigned long long t = blockIdx.x; t < nfb; t += gridDim.x) {
        const unsigned long long iters0 = iters;
        const int i = __builtin_amdgcn_readfirstlane(fb_list[t]);
        const double4 pi = pos[i];
        const double xi[3] = {uniform_d(pi.x), uniform_d(pi.y), uniform_d(pi.z)};
        // residual and slope at H, summing over r < H
        auto eval = [&](double H, double& f, double& fp, double& nk) {
            const double H2 = H * H, iH = 1.0 / H;
            double s = 0.0, sq = 0.0;
            scan_cells(td, tab, pos, S, lane, xi, xi, H + pd, [&](const double4& q, bool valid, int, int wrap) {
                const double r2 = sq_disp(q, xi, wrap, td.box);
                if (valid && r2 < H2) {
                    const double qq = sqrt(r2) * iH;
                    s += spline_w(qq);
                    sq += spline_qdw(qq);
                }
            });
            wave_sum2_d(s, sq, s, sq);
            f = c32 * s - ph.n_ngb;
            fp = -c32 * sq * iH;
            nk = kernel_norm(H) * s;
        };
        double lo = 0.0, hi = a.H[i];
        hi = uniform_d(hi);
        double f, fp, nk;
        bool ok = false;
        for (int k = 0; k < 64; k++) {
            iters++;
            if (!(hi < half)) hi = half * (1.0 - 1e-12);
            eval(hi, f, fp, nk);
            if (f >= 0.0) {
                ok = true;
                break;
            }
            if (!(hi < half * (1.0 - 1e-13))) break;
            lo = hi;
            hi *= 1.3;
        }
        bool conv = false;
        double Hc = hi;
        if (ok) {
            Hc = 0.5 * (lo + hi);
            for (int it = 0; it < ph.h_maxit; it++) {
                iters++;
                eval(Hc, f, fp, nk);
                if (newton_step(f, fp, lo, hi, Hc)) {
                    conv = true;
                    break;
                }
            }
        }
        int c = 0;
        if (ok && conv) {
            eval(Hc, f, fp, nk);
            const double H2 = Hc * Hc;
            const int cap = ph.max_ngb;
            // every gather neighbour but the particle itself, in scan order
            scan_cells(td, tab, pos, S, lane, xi, xi, Hc + pd, [&](const double4& q, bool valid, int, int wrap) {
                const double r2 = sq_disp(q, xi, wrap, td.box);
                const int j = (int)__double_as_longlong(q.w);
                const bool in = valid && r2 < H2 && j != i && sqrt(r2) < Hc;
                const unsigned long long b = __ballot(in);
                const int slot = c + __popcll(b & ((1ull << lane) - 1ull));
                if (in && slot < cap) jl[(long long)slot * n + i] = j;
                c += __popcll(b);
            });
            if (c > cap) {
                c = cap;
                over = 1;
                if (lane == 0) flag_index(cnt, i);
            }
        } else {
            nk = 0.0;
            if (!ok) noimg = 1;
            else noconv = 1;
            if (lane == 0) flag_index(cnt, i);
        }
        if (lane == 0) {
            a.H[i] = Hc;
            a.nk[i] = nk;
            a.V[i] = 1.0 / nk;
            gcount[i] = c;
            counts[i] = 0;
        }
        iters_max = max(iters_max, iters - iters0);
    }
    if (lane == 0) {
        if (iters) atomicAdd(&cnt->h_iters, iters);
        if (iters_max) atomicMax(&cnt->h_iters_max, iters_max);
        if (noconv) atomicAdd(&cnt->noconv, noconv);
        if (noimg) atomicAdd(&cnt->minimage, noimg);
        if (over) atomicAdd(&cnt->overflow, over);
    }
}

// Hierarchical steps with active subsets: a particle that keeps its kernel
// length and has an active particle within reach (mode kModeKept) lists its
// gather set r < H at the current positions with the scan and the distance
// test of the kernel-length solve, so that both particles of a pair decide on
// the same distance.  The lanes of a wave (Morton neighbours) scan together
// in the classes of the kernel-length scan.
__global__ __launch_bounds__(256) void k_gather_kept(PassArrays a, TreeDesc td, const int2* __restrict__ tab,
                                                     const double4* __restrict__ pos, Phys ph,
                                                     const unsigned char* __restrict__ mode, const double* __restrict__ pad,
                                                     int* __restrict__ jl, int* __restrict__ gcount,
                                                     int* __restrict__ counts) {
    __shared__ GroupLds lds[256 / kWave];
    GroupLds& S = lds[threadIdx.x / kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int i = xcd_block() * 256 + threadIdx.x;
    const bool sel = i < a.n && mode[i] == kModeKept;
    if (__ballot(sel) == 0) return;   // uniform over the wave
    const long long n = a.n;
    double xi[3] = {0.0, 0.0, 0.0};
    double H = 0.0;
    if (sel) {
        const double4 p = pos[i];
        xi[0] = p.x;
        xi[1] = p.y;
        xi[2] = p.z;
        H = a.H[i];
    }
    // scanned a little beyond H, so that no r < H is lost to the rounding of r^2
    const double Rs = H * (1.0 + 1e-9);
    const int cap = ph.max_ngb;
    int c = 0;
    bool need = sel && Rs > 0.0;
    for (int pass = 0; pass < kWave && __ballot(need); pass++) {
        const ScanClass cl = scan_class(need, Rs, xi);
        group_scan<true>(td, tab, pos, S, lane, cl.bmin, cl.bmax, cl.Rq, *pad, xi, Rs * Rs, cl.in, [&](int j, double r2) {
            const double r = sqrt_mid(r2);
            if (r < H && j != i) {
                if (c < cap) jl[(long long)c * n + i] = j;
                c++;
            }
        });
        need = need && !cl.in;
    }
    if (sel) {
        gcount[i] = min(c, cap);
        counts[i] = max(c - cap, 0);   // beyond cap: an overflow, counted when the tails are sorted
    }
}

// --------------------------------------------------------------- flux lists
// The flux set r < max(H_i, H_j) is the gather set of i plus every j that has
// i in its gather set with r >= H_i.  The gradient kernel, which walks every
// gather list anyway, appends each such j to i's list (atomic slot); then each
// list sorts its appended tail by index so the list, and every sum over it, is
// deterministic.
constexpr int kTailNet = 32;   // tails up to this length are sorted in registers

// Tail entries travel in bins, one per 256 consecutive particles: an entry is
// (i, j mod 256), appended to j's bin by whoever met the pair.  A wave's
// appends go to a few bins, so it takes one atomic per bin and writes runs of
// entries, where an atomic and a 4-byte store per entry, each to a line of its
// own, cost the gradient kernel 5.7 of its 14 ms (clustered 16.8M).  What a bin
// cannot hold is counted per particle in counts and put at the end of the
// particle's list slots, from the last one down.
struct Bins {
    int2* entry;    // kBinEntries per particle
    int* fill;      // entries per bin (appended ones, which may exceed what it holds)
};
__device__ __forceinline__ int bin_room(int bin, int n) { return kBinEntries * min(256, n - (bin << 8)); }
__device__ __forceinline__ void bin_store(const Bins& bins, int* __restrict__ counts, int* __restrict__ list,
                                          const int* __restrict__ gcount, int cap, int n, int j, int at, int i) {
    const int bin = j >> 8;
    if (at < bin_room(bin, n)) {
        bins.entry[(long long)bin * (256 * kBinEntries) + at] = make_int2(i, j & 255);
    } else {
        const int s = atomicAdd(&counts[j], 1);
        if (gcount[j] + s < cap) list[(long long)(cap - 1 - s) * n + j] = i;
    }
}
// one append by the calling lane alone
__device__ __forceinline__ void bin_append(const Bins& bins, int* __restrict__ counts, int* __restrict__ list,
                                           const int* __restrict__ gcount, int cap, int n, int j, int i) {
    bin_store(bins, counts, list, gcount, cap, n, j, atomicAdd(&bins.fill[j >> 8], 1), i);
}

// bitonic sorting network on N registers (indices fixed at compile time)
template <int N>
__device__ __forceinline__ void bitonic_net(int* v) {
#pragma unroll
    for (int w = 2; w <= N; w <<= 1)
#pragma unroll
        for (int h = w >> 1; h > 0; h >>= 1)
#pragma unroll
            for (int k = 0; k < N; k++) {
                const int l = k ^ h;
                if (l > k) {
                    const int lo_v = min(v[k], v[l]), hi_v = max(v[k], v[l]);
                    const bool up = (k & w) == 0;
                    v[k] = up ? lo_v : hi_v;
                    v[l] = up ? hi_v : lo_v;
                }
            }
}

// The tails of a block's 256 particles, from their bin: the entries are dealt to
// their particles in LDS, sorted by index and written behind the gather parts,
// so every later sum over a list runs in one order; counts[i] becomes the length
// of the whole list.  A short tail is sorted in registers by a network sized to
// the wave's longest such tail, and written through its LDS column a row at a
// time (the list is interleaved, list[k * n + i], and tails start at different
// rows), each store one coalesced row segment of the wave's columns.  Longer
// tails, and those with entries that the bin could not hold, are ranked by the
// whole wave in LDS.
__global__ __launch_bounds__(256) void k_sort_tails(int n, int cap, const int* __restrict__ gcount,
                                                     int* __restrict__ counts, int* __restrict__ list, Bins bins,
                                                     Counters* cnt) {
    cnt = counter_copy(cnt);
    __shared__ int col[kTailNet][256];
    __shared__ int dealt[256], gathered[256];
    const int bin = xcd_block();
    const int i = bin * 256 + threadIdx.x;
    unsigned long long c = 0, over = 0, gsum = 0;
    int g = 0, t = 0, extra = 0;
    if (i < n) {
        g = gcount[i];
        extra = counts[i];
    }
    dealt[threadIdx.x] = 0;
    gathered[threadIdx.x] = g;
    __syncthreads();
    const int fill = min(bins.fill[bin], bin_room(bin, n));
    const int2* __restrict__ entry = bins.entry + (long long)bin * (256 * kBinEntries);
    for (int e = threadIdx.x; e < fill; e += 256) {
        const int2 x = entry[e];
        const int s = atomicAdd(&dealt[x.y], 1);
        if (s < kTailNet) col[s][x.y] = x.x;
        else if (gathered[x.y] + s < cap) list[(long long)(gathered[x.y] + s) * n + bin * 256 + x.y] = x.x;
    }
    __syncthreads();
    const int from_bin = dealt[threadIdx.x];
    if (i < n) {
        gsum = (unsigned long long)g;
        int e = g + from_bin + extra;
        c = (unsigned long long)e;
        if (e > cap) {
            over = 1;
            flag_index(cnt, i);
            e = cap;
        }
        counts[i] = e;
        t = e - g;
    }
    const bool net = t > 0 && t <= kTailNet && extra == 0;
    const int tmax = wave_max_i(net ? t : 0);
    if (tmax > 0) {
        int v[kTailNet];
#pragma unroll
        for (int k = 0; k < kTailNet; k++) v[k] = net && k < t ? col[k][threadIdx.x] : INT_MAX;
        if (tmax <= 8) bitonic_net<8>(v);
        else if (tmax <= 16) bitonic_net<16>(v);
        else bitonic_net<kTailNet>(v);
#pragma unroll
        for (int k = 0; k < kTailNet; k++)
            if (k < t && net) col[k][threadIdx.x] = v[k];
        const int rlo = wave_min_i(net ? g : INT_MAX);
        const int rhi = wave_max_i(net ? g + t : INT_MIN);
        for (int r = rlo; r < rhi; r++)
            if (net && r >= g && r < g + t) list[(long long)r * n + i] = col[r - g][threadIdx.x];
    }
    if (t > 0 && !net) {
        // the whole tail into its slots: what was dealt to the column, and the
        // entries at the end of the particle's slots (moved down in order)
        for (int k = 0; k < min(kTailNet, min(from_bin, t)); k++) list[(long long)(g + k) * n + i] = col[k][threadIdx.x];
        const int kept = min(extra, cap - g);
        for (int k = 0; k < kept && from_bin + k < t; k++)
            list[(long long)(g + from_bin + k) * n + i] = list[(long long)(cap - kept + k) * n + i];
    }
    // Long tails, one at a time per wave: the tail goes to a contiguous LDS
    // region of the wave, every lane ranks its entries against all of them (ties,
    // which a list does not hold, by position) and writes each entry to its slot.
    __syncthreads();   // every wave is done with the columns, and the moves above are visible
    int* wb = &col[0][0] + (threadIdx.x >> 6) * (kTailNet * kWave);
    const int lane = threadIdx.x & (kWave - 1);
    unsigned long long lm = __ballot(t > 0 && !net && t <= kTailNet * kWave);
    while (lm) {
        const int src = __ffsll((long long)lm) - 1;
        lm &= lm - 1;
        const int gs = __shfl(g, src, kWave), ts = __shfl(t, src, kWave), is = __shfl(i, src, kWave);
        for (int k = lane; k < ts; k += kWave) wb[k] = list[(long long)(gs + k) * n + is];
        wave_lds_sync();
        for (int k = lane; k < ts; k += kWave) {
            const int v = wb[k];
            int rank = 0;
            for (int q = 0; q < ts; q++) {
                const int u = wb[q];
                rank += (u < v || (u == v && q < k)) ? 1 : 0;
            }
            list[(long long)(gs + rank) * n + is] = v;
        }
        wave_lds_sync();   // the next tail overwrites the region
    }
    if (t > kTailNet * kWave) {
        // beyond what the wave's LDS region holds: sort in place
        for (int k = g + 1; k < g + t; k++) {
            const int v = list[(long long)k * n + i];
            int q = k - 1;
            while (q >= g && list[(long long)q * n + i] > v) {
                list[(long long)(q + 1) * n + i] = list[(long long)q * n + i];
                q--;
            }
            list[(long long)(q + 1) * n + i] = v;
        }
    }
    count_add(&cnt->list_entries, c);
    count_add(&cnt->gather_entries, gsum);
    count_max(&cnt->list_max, c);
    count_add(&cnt->overflow, over);
}

// ---------------------------------------------------------------- gradients
// Record of one particle for the flux kernel (32 slots, one or two cache lines):
// 0-2 x, y, z (FP64 record; the FP32 record holds the FP64 pressure in 0-1) | 3 1/H | 4 K = V^2 8/(pi H^3) | 5 rho | 6 P | 7-9 v | 10-15 B |
// 16-30 grad | 31 c.  With 1/H and K per particle a face needs no division for its kernel weights:
// V^2 W(r, H) = K w(r/H).
enum { R_X = 0, R_IH = 3, R_K = 4, R_RHO = 5, R_P = 6, R_V0 = 7, R_B = 10, R_G = 16, R_C = 31 };

// What the gradient kernel reads of a neighbour, packed into one 128-byte line
// per particle: (x, y, z, H), (rho, vx, vy, vz), (P, -, -, -), unused.
__device__ __forceinline__ void pack_values(const PassArrays& a, const Phys& ph, int i, double v[9]) {
    v[0] = a.x[i];
    v[1] = a.y[i];
    v[2] = a.z[i];
    v[3] = a.H[i];
    const double rho = a.m[i] * a.nk[i];
    v[4] = rho;
    v[5] = a.vx[i];
    v[6] = a.vy[i];
    v[7] = a.vz[i];
    v[8] = (ph.gamma - 1.0) * rho * a.u[i];
}
__device__ __forceinline__ void pack_one(const PassArrays& a, const Phys& ph, double4* __restrict__ prim, int i) {
    double v[9];
    pack_values(a, ph, i, v);
    prim[4 * (long long)i + 0] = make_double4(v[0], v[1], v[2], v[3]);
    prim[4 * (long long)i + 1] = make_double4(v[4], v[5], v[6], v[7]);
    prim[4 * (long long)i + 2] = make_double4(v[8], 0.0, 0.0, 0.0);
}

// (the pack kernels run in blocks of 256 and empty the blocks' tail bins)
// The records leave through LDS in whole 128-byte lines, as the flux records do:
// bounded by memory, 10 loads and 128 bytes of stores a particle.  Stored by each
// thread, 96 bytes every 128 reached memory as partial lines.  Measured: 2.1M
// particles 138 -> 74 us, 16.8M 1.33 -> 0.61 ms.
__global__ __launch_bounds__(256) void k_pack_prim(PassArrays a, Phys ph, double4* __restrict__ prim,
                                                   int* __restrict__ fill) {
    __shared__ TeamLds<8> lds[256 / kWave];
    TeamLds<8>& S = lds[threadIdx.x / kWave];
    const int lane = threadIdx.x % kWave;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (threadIdx.x == 0) fill[blockIdx.x] = 0;
    const bool act = i < a.n;
    const unsigned long long lanes = __ballot(act);
    double v[16] = {};
    if (act) pack_values(a, ph, i, v);
#pragma unroll
    for (int c = 0; c < 8; c++) {
        uint4 u;
        __builtin_memcpy(&u, v + 2 * c, 16);
        team_put(S, c, lane, u);
    }
    wave_lds_sync();
    team_store<128>(S, (char*)prim + (size_t)(unsigned)(i - lane) * 128, lanes, lane);
}

// A boundary with active subsets reads the records of the active particles'
// gather neighbours (their gradients) and of the active particles themselves
// (the kept particles' tail appends) only: each active particle packs its own
// and its gather neighbours' records.  A record packed by several of them gets
// the same values from each.  The others keep stale records, which no kernel
// of that boundary reads.
__global__ void k_pack_prim_active(PassArrays a, Phys ph, const int* __restrict__ gcount,
                                   const unsigned char* __restrict__ mode, const int* __restrict__ list,
                                   double4* __restrict__ prim, int* __restrict__ fill) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (threadIdx.x == 0) fill[blockIdx.x] = 0;
    if (i >= a.n || mode[i] != kModeSolve) return;
    const long long n = a.n;
    pack_one(a, ph, prim, i);
    const int cnum = gcount[i];
    for (int k = 0; k < cnum; k++) pack_one(a, ph, prim, list[(long long)k * n + i]);
}

// One wave per block; the neighbours' records come by lane teams, and while one is
// summed the next is on its way to LDS.  The tail appends of the wave queue in LDS
// until the sums are done: in the loop a wave had an atomic's round trip to L2 in
// nearly every step.  Then the queue is worked off 64 at a time, four rounds in
// flight; the entries of a round that go to one bin take their places with one
// atomic.  The flux records leave through LDS too, in whole 128-byte lines: 16-byte
// stores 256 bytes apart reached memory as partial lines.  Three waves per SIMD: the
// sums, the record in hand and the loop's values take 140 VGPRs, and a fourth wave
// spills.  Measured: lattice 2.1M 1.06 -> 0.81 ms, clustered 16.8M 13.8 -> 9.2 ms,
// shock tube 295k (mixed) 0.177 -> 0.114 ms.
// With HIER (hierarchical steps with active subsets) only the particles of
// mode kModeSolve get new gradients; a kept particle with a gather list only
// appends itself to the lists of its active neighbours that do not reach it.
// A particle's list is shared by SPLIT lanes, 64 / SPLIT apart, whose sums meet
// at the end: with one lane a particle, a set of 32,768 is 512 waves for 1,024
// SIMDs, each as long as its longest list.  Up to kGradSplit4 particles four
// lanes, up to kGradSplit2 two; beyond, where the waves fill the chip, one
// (the sums of E stay in the order of the list, which the gradient matrices of
// ill-conditioned particles show).  Measured, one / two / four / eight lanes:
// lattice 4,096 36 / 23 / 18 / 18 us, 32,768 39 / 31 / 29 / 39, 64,000 48 / 38 /
// 42 / 52, 110,592 53 / 54 / 57 / 78; clustered 32,768 182 / 92 / 54 / 51,
// 64,000 293 / 117 / 73 / 63, 110,592 158 / 95 / 79 / 86.
constexpr int kGradSplit4 = 65536;
constexpr int kGradSplit2 = 131072;
constexpr int kGradWaves = 3;
constexpr int kAppends = 768;   // appends a wave holds back
struct GradLds {
    TeamLds<8> t;
    int to[kAppends];               // particle j whose list takes ...
    unsigned char from[kAppends];   // ... the particle of this lane
};
template <bool MIXED, bool HIER, int SPLIT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kGradWaves))) void k_gradients(PassArrays a, Phys ph, const int* __restrict__ gcount,
                                                    int* __restrict__ counts, int* __restrict__ list, Bins bins,
                                                    const double4* __restrict__ prim, void* __restrict__ recp,
                                                    Counters* cnt, const unsigned char* __restrict__ mode,
                                                    const long long* __restrict__ home) {
    cnt = counter_copy(cnt);
    __shared__ GradLds lds;
    TeamLds<8>& S8 = lds.t;
    static_assert(!HIER || SPLIT == 1, "one lane per particle with active subsets");
    constexpr int kOwn = kWave / SPLIT;   // particles of the wave
    const int lane = threadIdx.x, sub = lane / kOwn;
    const int i = xcd_block() * kOwn + lane % kOwn;
    if (HIER && i < a.n && mode[i] == kModeKept) {
        const long long n = a.n;
        const double xi[3] = {a.x[i], a.y[i], a.z[i]};
        const int cnum = gcount[i];
        for (int k = 0; k < cnum; k++) {
            const int j = list[(long long)k * n + i];
            if (mode[j] != kModeSolve) continue;   // the pair is not due (and j's record may be stale)
            const double4 pj = prim[4 * (long long)j + 0];
            double d[3];
            displacement(ph, xi, pj.x, pj.y, pj.z, d);
            const double r = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
            if (!(r < pj.w)) bin_append(bins, counts, list, gcount, ph.max_ngb, a.n, j, i);
        }
    }
    const bool act = i < a.n && (!HIER || mode[i] == kModeSolve);
    unsigned long long ill = 0, nonfin = 0, condbits = 0;
    const long long n = a.n;
    double xi[3] = {0.0, 0.0, 0.0}, phi_i[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    double Hi = 1.0, Vi = 1.0;
    int cnum = 0;
    if (act) {
        xi[0] = a.x[i];
        xi[1] = a.y[i];
        xi[2] = a.z[i];
        Hi = a.H[i];
        Vi = a.V[i];
        phi_i[0] = a.m[i] * a.nk[i];
        phi_i[1] = a.vx[i];
        phi_i[2] = a.vy[i];
        phi_i[3] = a.vz[i];
        phi_i[4] = (ph.gamma - 1.0) * phi_i[0] * a.u[i];
        cnum = gcount[i];
    }
    const double rho_i = phi_i[0], P_i = phi_i[4];
    double E[6] = {0, 0, 0, 0, 0, 0};
    double S[15];
    double pmax[5], pmin[5];
#pragma unroll
    for (int k = 0; k < 15; k++) S[k] = 0.0;
#pragma unroll
    for (int f = 0; f < 5; f++) pmax[f] = pmin[f] = phi_i[f];
    double rmax = 0.0;
    const double norm = kernel_norm(Hi), iH = 1.0 / Hi;
    const float normf = (float)norm, iHf = (float)iH;
    const int cap = ph.max_ngb;
    const int self = i < a.n ? i : a.n - 1;   // a record to load where a lane has no neighbour
    const int kmax = __builtin_amdgcn_readfirstlane(wave_max_i((cnum + SPLIT - 1) / SPLIT));
    auto entry = [&](int k) {
        const int e = k * SPLIT + sub;
        return e < cnum ? list[(long long)e * n + i] : -1;
    };
    int j = entry(0), jn = entry(1);
    int napp = 0;   // appends of the wave so far
    const unsigned long long below = (1ull << lane) - 1ull;
    if (kmax > 0) team_load<128, 5>(S8, prim, a.n, j >= 0 ? j : self, lane);
    for (int k = 0; k < kmax; k++) {
        wait_vmem();
        wave_lds_sync();
        double rec[10];   // x, y, z, H, rho, vx, vy, vz, P
#pragma unroll
        for (int c = 0; c < 5; c++) {
            const uint4 u = team_chunk(S8, c, lane);
            __builtin_memcpy(rec + 2 * c, &u, 16);
        }
        const int jc = j;
        j = jn;
        wave_lds_sync();
        wait_lds();
        if (k + 1 < kmax) team_load<128, 5>(S8, prim, a.n, j >= 0 ? j : self, lane);
        jn = entry(k + 2);
        double d[3];
        displacement(ph, xi, rec[0], rec[1], rec[2], d);
        const double r = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
        const bool append = jc >= 0 && !(r < rec[3]);
        const unsigned long long am = __ballot(append);
        if (append) {
            const int at = napp + __popcll(am & below);
            if (at < kAppends) {
                lds.to[at] = jc;
                lds.from[at] = (unsigned char)lane;
            } else {
                bin_append(bins, counts, list, gcount, cap, a.n, jc, i);
            }
        }
        napp += __popcll(am);
        if (jc < 0) continue;
        const double* phi_j = rec + 4;
        // MIXED: the pairwise kernel weight in FP32; the moments and sums in FP64, so
        // that E and the gradient sums share one set of weights and the
        // conditioning of E does not amplify per-product rounding
        const double psi = MIXED ? (double)(normf * spline_w((float)r * iHf)) * Vi : norm * spline_w(r * iH) * Vi;
        E[0] += d[0] * d[0] * psi;
        E[1] += d[0] * d[1] * psi;
        E[2] += d[0] * d[2] * psi;
        E[3] += d[1] * d[1] * psi;
        E[4] += d[1] * d[2] * psi;
        E[5] += d[2] * d[2] * psi;
#pragma unroll
        for (int f = 0; f < 5; f++) {
            const double df = (phi_j[f] - phi_i[f]) * psi;
            S[3 * f + 0] += df * d[0];
            S[3 * f + 1] += df * d[1];
            S[3 * f + 2] += df * d[2];
        }
#pragma unroll
        for (int f = 0; f < 5; f++) {
            pmax[f] = fmax(pmax[f], phi_j[f]);
            pmin[f] = fmin(pmin[f], phi_j[f]);
        }
        rmax = fmax(rmax, r);
    }
    {
        const int held = min(napp, kAppends), r0 = i - lane % kOwn;
        wave_lds_sync();
        for (int b = 0; b < held; b += 4 * kWave) {
            int to[4], lead[4], rank[4], at[4];
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const int e = b + q * kWave + lane;
                to[q] = e < held ? lds.to[e] : -1;
                lead[q] = lane;
                rank[q] = 0;
                int share = 0;   // appends of the round that go to the lane's bin
                unsigned long long left = __ballot(to[q] >= 0);
                while (left) {
                    const int first = __ffsll((long long)left) - 1;
                    const int bin = __builtin_amdgcn_readlane(to[q], first) >> 8;
                    const bool same = (to[q] >> 8) == bin;   // (-1 >> 8 is no bin)
                    const unsigned long long m = __ballot(same);
                    if (same) {
                        lead[q] = first;
                        rank[q] = __popcll(m & below);
                        share = __popcll(m);
                    }
                    left &= ~m;
                }
                at[q] = to[q] >= 0 && lead[q] == lane ? atomicAdd(&bins.fill[to[q] >> 8], share) : 0;
            }
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const int base = __shfl(at[q], lead[q], kWave);
                if (to[q] >= 0)
                    bin_store(bins, counts, list, gcount, cap, a.n, to[q], base + rank[q],
                              r0 + lds.from[b + q * kWave + lane] % kOwn);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < 6; k++) split_sum<SPLIT>(E[k]);
#pragma unroll
    for (int k = 0; k < 15; k++) split_sum<SPLIT>(S[k]);
#pragma unroll
    for (int f = 0; f < 5; f++) {
        split_max<SPLIT>(pmax[f]);
        split_min<SPLIT>(pmin[f]);
    }
    split_max<SPLIT>(rmax);
    const bool own = act && sub == 0;
    // (lanes without a particle run along on zeros and store nothing)
    {
        // B = E^-1 by cofactors (E symmetric: xx xy xz yy yz zz)
        const double c00 = E[3] * E[5] - E[4] * E[4];
        const double c01 = E[2] * E[4] - E[1] * E[5];
        const double c02 = E[1] * E[4] - E[2] * E[3];
        const double c11 = E[0] * E[5] - E[2] * E[2];
        const double c12 = E[1] * E[2] - E[0] * E[4];
        const double c22 = E[0] * E[3] - E[1] * E[1];
        const double det = E[0] * c00 + E[1] * c01 + E[2] * c02;
        const double idet = 1.0 / det;
        const double B[6] = {c00 * idet, c01 * idet, c02 * idet, c11 * idet, c12 * idet, c22 * idet};
        const double fe = E[0] * E[0] + E[3] * E[3] + E[5] * E[5] + 2.0 * (E[1] * E[1] + E[2] * E[2] + E[4] * E[4]);
        const double fb = B[0] * B[0] + B[3] * B[3] + B[5] * B[5] + 2.0 * (B[1] * B[1] + B[2] * B[2] + B[4] * B[4]);
        const double cond = sqrt(fe) * sqrt(fb);
        if (own && (!(det > 0.0) || !(cond <= ph.cond_max))) {
            ill = 1;
            flag_index(cnt, i);
        }
        if (own && cond > 0.0) condbits = __double_as_longlong(cond);
        // the limiter constant: beta, or with the optional limiters (R24) beta moved
        // towards beta_min linearly in log10(cond) between cond_lo and cond_hi
        double beta = ph.beta;
        if (ph.limiter) {
            double t;
            if (cond <= ph.cond_lo) t = 0.0;
            else if (cond < ph.cond_hi) t = (log10(cond) - log10(ph.cond_lo)) / (log10(ph.cond_hi) - log10(ph.cond_lo));
            else t = 1.0;
            beta = ph.beta + (ph.beta_min - ph.beta) * t;
        }
        double g[15];
        double al[5];
        const double half = 0.5 * rmax;
#pragma unroll
        for (int f = 0; f < 5; f++) {
            const double* s = S + 3 * f;
            const double g0 = B[0] * s[0] + B[1] * s[1] + B[2] * s[2];
            const double g1 = B[1] * s[0] + B[3] * s[1] + B[4] * s[2];
            const double g2 = B[2] * s[0] + B[4] * s[1] + B[5] * s[2];
            double alpha;
            if (!MIXED) {
                const double gn = sqrt(g0 * g0 + g1 * g1 + g2 * g2);
                alpha = 1.0;
                if (gn > 0.0) {
                    const double up = (pmax[f] - phi_i[f]) / (gn * half);
                    const double dn = (phi_i[f] - pmin[f]) / (gn * half);
                    alpha = fmin(1.0, beta * fmin(up, dn));
                }
            } else {
                const float h0 = (float)g0, h1 = (float)g1, h2 = (float)g2;
                const float gn = sqrtf(h0 * h0 + h1 * h1 + h2 * h2);
                float af = 1.0f;
                if (gn > 0.0f) {
                    const float hf = (float)half;
                    const float up = (float)(pmax[f] - phi_i[f]) / (gn * hf);
                    const float dn = (float)(phi_i[f] - pmin[f]) / (gn * hf);
                    af = fminf(1.0f, (float)beta * fminf(up, dn));
                }
                alpha = (double)af;
            }
            al[f] = alpha;
            g[3 * f + 0] = alpha * g0;
            g[3 * f + 1] = alpha * g1;
            g[3 * f + 2] = alpha * g2;
        }
        if (own) {
            const long long io = HIER ? home[i] : i;   // column of B, grad and alpha
#pragma unroll
            for (int k = 0; k < 6; k++) a.B[k * n + io] = B[k];
#pragma unroll
            for (int k = 0; k < 15; k++) {
                a.grad[k * n + io] = g[k];
                if (!isfinite(g[k])) nonfin = 1;
            }
            if (a.alpha) {
#pragma unroll
                for (int f = 0; f < 5; f++) a.alpha[f * n + io] = al[f];
            }
            a.rho[i] = rho_i;
            a.P[i] = P_i;
        }
        const double c_i = sqrt(ph.gamma * P_i / rho_i);
        using T = typename std::conditional<MIXED, float, double>::type;
        T v[32];
        if constexpr (!MIXED) {
            v[0] = xi[0];
            v[1] = xi[1];
            v[2] = xi[2];
        } else {
            // slots 0-1: the pressure in FP64 (its two halves), for the pressure
            // difference across a face; slot 2 unused
            const long long pbits = __double_as_longlong(P_i);
            v[0] = __int_as_float((int)(pbits & 0xffffffffll));
            v[1] = __int_as_float((int)(pbits >> 32));
            v[2] = 0.0f;
        }
        v[R_IH] = (T)iH;
        v[R_K] = (T)(Vi * Vi * norm);
        v[R_RHO] = (T)rho_i;
        v[R_P] = (T)P_i;
#pragma unroll
        for (int c = 0; c < 3; c++) v[R_V0 + c] = (T)phi_i[1 + c];
#pragma unroll
        for (int k = 0; k < 6; k++) v[R_B + k] = (T)B[k];
#pragma unroll
        for (int k = 0; k < 15; k++) v[R_G + k] = (T)g[k];
        v[R_C] = (T)c_i;
        // the wave's records, 128 bytes of each at a time, transposed in LDS: eight
        // lanes then store one record's line
        const unsigned long long stored = __ballot(own);
#pragma unroll
        for (int h = 0; h < (int)sizeof(T) / 4; h++) {
            wave_lds_sync();
#pragma unroll
            for (int c = 0; c < 8; c++) {
                uint4 u;
                __builtin_memcpy(&u, v + (8 * h + c) * (16 / sizeof(T)), 16);
                team_put(S8, c, lane, u);
            }
            wave_lds_sync();
            team_store<32 * sizeof(T)>(S8, (char*)recp + (size_t)(unsigned)(i - lane % kOwn) * (32 * sizeof(T)) + 128 * h,
                                       stored, lane);
        }
    }
    count_add(&cnt->illcond, ill);
    count_add(&cnt->nonfinite, nonfin);
    count_max(&cnt->cond_bits, condbits);
}

// Hierarchical steps with active subsets: the records of the particles that
// keep their kernel length and gradients and take part in a due pair (a flux
// list), from their kept H, V, n, B and limited gradients (B and grad at
// column home[i]) with the current position and predicted state, as the
// gradient kernel writes them.
__global__ void k_pack_rec_kept(PassArrays a, Phys ph, const unsigned char* __restrict__ mode,
                                const long long* __restrict__ home, const int* __restrict__ counts,
                                double* __restrict__ recp) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.n || mode[i] == kModeSolve || counts[i] == 0) return;
    const long long n = a.n;
    const long long h = home[i];
    const double Hi = a.H[i], Vi = a.V[i];
    const double rho_i = a.m[i] * a.nk[i];
    const double P_i = (ph.gamma - 1.0) * rho_i * a.u[i];
    double v[32];
    v[0] = a.x[i];
    v[1] = a.y[i];
    v[2] = a.z[i];
    v[R_IH] = 1.0 / Hi;
    v[R_K] = Vi * Vi * kernel_norm(Hi);
    v[R_RHO] = rho_i;
    v[R_P] = P_i;
    v[R_V0 + 0] = a.vx[i];
    v[R_V0 + 1] = a.vy[i];
    v[R_V0 + 2] = a.vz[i];
#pragma unroll
    for (int k = 0; k < 6; k++) v[R_B + k] = a.B[k * n + h];
#pragma unroll
    for (int k = 0; k < 15; k++) v[R_G + k] = a.grad[k * n + h];
    v[R_C] = sqrt(ph.gamma * P_i / rho_i);
    double2* r2 = (double2*)(recp + (long long)i * 32);
#pragma unroll
    for (int k = 0; k < 16; k++) r2[k] = make_double2(v[2 * k], v[2 * k + 1]);
}

// ------------------------------------------------------------------- fluxes
template <typename T>
struct PairOut {
    T Fm;
    T Fp[3];
    T FE;
    int fallback, clamp;
};

template <typename T>
__device__ __forceinline__ T tsqrt(T v);
template <>
__device__ __forceinline__ double tsqrt<double>(double v) { return sqrt(v); }
template <>
__device__ __forceinline__ float tsqrt<float>(float v) { return sqrtf(v); }

// One unordered pair in canonical order (the lower index is the left state),
// evaluated by the owner `m` of one side with the record `o` of the other; mL
// says whether m is the left side, d = x_R - x_L is the canonical displacement
// and r its length.  Every per-side quantity is written with one expression
// for that side (left: +1/2, right: -1/2 along d), and the sum of the two
// face halves is commutative and unfused, so both owners produce the same
// bits; only the reconstructed face states are put in left/right order.
// MFV (the finite-volume form): the full HLLC flux through the face, which
// moves with w.  Only the side that the star-state selection picks is built:
// K is the left side when S* >= 0 (or S_L >= 0), else the right side, and the
// star correction S_K (U*_K - U_K) is added unless that side's outer wave has
// already passed the face.  In the face frame (primes) the side state is
// rho, v' = v - w, E = P/(gamma-1) + rho |v'|^2/2, with physical flux
// (rho u, rho u v' + P n, (E + P) u), u = v'.n; its star state scales by
// f = rho (S_K - u)/(S_K - S*) and takes the normal speed S*.  The lab-frame
// flux adds w times the mass flux to the momentum flux and
// w.F_mom' + |w|^2/2 F_mass to the energy flux.
template <typename T>
__device__ __forceinline__ void mfv_flux(const T qL[5], const T qR[5], const T w[3], const T nh[3], T uL, T uR,
                                         T SL, T SR, T Ss, T gamma, T Amag, PairOut<T>& out) {
    const bool left = (SL >= T(0)) || (Ss >= T(0));
    const bool star = left ? !(SL >= T(0)) : (SR >= T(0));
    T q[5];
#pragma unroll
    for (int f = 0; f < 5; f++) q[f] = left ? qL[f] : qR[f];
    const T u = left ? uL : uR;
    const T S = left ? SL : SR;
    const T rho = q[0], P = q[4];
    const T vp[3] = {q[1] - w[0], q[2] - w[1], q[3] - w[2]};
    const T E = P / (gamma - T(1)) + T(0.5) * rho * (vp[0] * vp[0] + vp[1] * vp[1] + vp[2] * vp[2]);
    T F[5];
    F[0] = rho * u;
#pragma unroll
    for (int c = 0; c < 3; c++) F[1 + c] = rho * vp[c] * u + P * nh[c];
    F[4] = (E + P) * u;
    if (star) {
        const T f = rho * (S - u) / (S - Ss);
        const T du = Ss - u;
        if (sizeof(T) == 8) {
            F[0] += S * (f - rho);
#pragma unroll
            for (int c = 0; c < 3; c++) F[1 + c] += S * (f * (vp[c] + du * nh[c]) - rho * vp[c]);
            F[4] += S * (f * (E / rho + du * (Ss + P / (rho * (S - u)))) - E);
        } else {
            // FP32: the same flux in the form S* U*_K + P*_K (0, n, S*), with the
            // side's star pressure P*_K = P + rho (S - u)(S* - u).  F_K +
            // S_K (U*_K - U_K) equals it identically (the star state satisfies the
            // jump conditions across S_K), but subtracts terms much larger than a
            // slow face's mass flux; this form has no such cancellation.
            const T Pst = P + rho * (S - u) * du;
            F[0] = f * Ss;
#pragma unroll
            for (int c = 0; c < 3; c++) F[1 + c] = f * (vp[c] + du * nh[c]) * Ss + Pst * nh[c];
            F[4] = (f * (E / rho + du * (Ss + P / (rho * (S - u)))) + Pst) * Ss;
        }
    }
    const T ww = w[0] * w[0] + w[1] * w[1] + w[2] * w[2];
    out.Fm = F[0] * Amag;
#pragma unroll
    for (int c = 0; c < 3; c++) out.Fp[c] = (F[1 + c] + w[c] * F[0]) * Amag;
    out.FE = (F[4] + w[0] * F[1] + w[1] * F[2] + w[2] * F[3] + T(0.5) * ww * F[0]) * Amag;
}

// The optional pairwise limiter (R23) on one side's face value f, with pk that
// side's centre value and po the other's: on the other particle's side at most
// D/4 past the midpoint interpolant, on its own side at most D/2 outside the
// centre range [lo, hi] (D = hi - lo); a widened bound that would not keep the
// sign is lo / (1 + D / (2|lo|)) (hi likewise), taken here as
// lo |lo| / (|lo| + D/2).  That bound only matters where the value passes it,
// which v (|lo| + D/2) against lo |lo| decides without dividing, so the
// division runs only when a lane of the wave clamps there.  Each owner
// evaluates it with the same arguments for the same side, so both copies of a
// pair agree bit for bit.
__device__ __forceinline__ double lim_min(double a, double b) { return fmin(a, b); }
__device__ __forceinline__ float lim_min(float a, float b) { return fminf(a, b); }
__device__ __forceinline__ double lim_max(double a, double b) { return fmax(a, b); }
__device__ __forceinline__ float lim_max(float a, float b) { return fmaxf(a, b); }

// In t = s f, with s = +1 where the side's own value is the lower of the two
// and -1 where it is the higher, both cases read as the first one: t at most
// s mid + D/4 and at least s pk - D/2 (the sign flips are exact), so the bound
// is two min/max instructions.
// The same bound in the direct form, for the FP32 records (where the
// sign-flipped form measured slower: 18.0 against 22.1 ms on the clustered set).
template <typename T>
__device__ __forceinline__ T pair_limit_direct(T f, T pk, T po) {
    if (pk == po) return pk;
    const bool below = pk < po;   // the side's own value is the lower one
    const T lo = below ? pk : po, hi = below ? po : pk;
    const T D = hi - lo;
    const T mid = T(0.5) * (pk + po);
    const T e = below ? lo : hi;
    const T wide = below ? lo - T(0.5) * D : hi + T(0.5) * D;
    const T inner = below ? mid + T(0.25) * D : mid - T(0.25) * D;
    T v = below ? (f < inner ? f : inner) : (f > inner ? f : inner);
    if (wide * e > T(0)) return below ? (v > wide ? v : wide) : (v < wide ? v : wide);
    const T ae = e < T(0) ? -e : e;
    const T den = ae + T(0.5) * D, num = e * ae;
    const bool clamp = below ? v * den < num : v * den > num;
    if (__ballot(clamp)) {
        if (clamp) v = num / den;
    }
    return v;
}

template <typename T>
__device__ __forceinline__ T pair_limit(T f, T pk, T po) {
    if constexpr (sizeof(T) == 4) return pair_limit_direct(f, pk, po);
    const T s = pk < po ? T(1) : T(-1);
    const T D = pk < po ? po - pk : pk - po;
    const T spk = s * pk;
    const T t = lim_min(s * f, s * (T(0.5) * (pk + po)) + T(0.25) * D);
    const T wide = spk - T(0.5) * D;
    const bool keep = wide * spk > T(0);
    T r = keep ? lim_max(t, wide) : t;
    // the sign-keeping bound s b = spk |pk| / (|pk| + D/2): clamp where t is below it
    const T apk = pk < T(0) ? -pk : pk;
    const T den = apk + T(0.5) * D, num = spk * apk;
    const bool clamp = !keep && t * den < num;
    if (__ballot(clamp)) {
        if (clamp) r = num / den;
    }
    return pk == po ? pk : s * r;
}

// the sound speeds sqrt(gp / rho) of the two sides; in FP64 as gp / sqrt(gp rho),
// one reciprocal square root in place of a division and a square root
__device__ __forceinline__ void sound_speeds(double gpL, double rL, double gpR, double rR, double& cL, double& cR) {
    const double xL = gpL * rL, xR = gpR * rR;
    if (__builtin_expect(is_mid(xL) && is_mid(xR), 1)) {
        sqrt_inv_mid(xL, cL);
        sqrt_inv_mid(xR, cR);
        cL *= gpL;
        cR *= gpR;
    } else {
        cL = sqrt(gpL / rL);
        cR = sqrt(gpR / rR);
    }
}
__device__ __forceinline__ void sound_speeds(float gpL, float rL, float gpR, float rR, float& cL, float& cR) {
    cL = sqrtf(gpL / rL);
    cR = sqrtf(gpR / rR);
}

template <typename T, bool MFV, bool LIM>
__device__ __forceinline__ PairOut<T> pair_flux(const T* __restrict__ m, const T* __restrict__ o, bool mL,
                                                const T d[3], T r, T gamma) {
    PairOut<T> out;
    out.Fm = out.Fp[0] = out.Fp[1] = out.Fp[2] = out.FE = T(0);
    out.fallback = out.clamp = 0;
    // face A = V_m^2 W_m B_m d + V_o^2 W_o B_o d (the kernel factor K = V^2 8/(pi H^3))
    const T km = m[R_K] * spline_w(r * m[R_IH]);
    const T ko = o[R_K] * spline_w(r * o[R_IH]);
    const T* Bm = m + R_B;
    const T* Bo = o + R_B;
    const T tm[3] = {Bm[0] * d[0] + Bm[1] * d[1] + Bm[2] * d[2], Bm[1] * d[0] + Bm[3] * d[1] + Bm[4] * d[2],
                     Bm[2] * d[0] + Bm[4] * d[1] + Bm[5] * d[2]};
    const T to[3] = {Bo[0] * d[0] + Bo[1] * d[1] + Bo[2] * d[2], Bo[1] * d[0] + Bo[3] * d[1] + Bo[4] * d[2],
                     Bo[2] * d[0] + Bo[4] * d[1] + Bo[5] * d[2]};
    T A[3];
#pragma unroll
    for (int c = 0; c < 3; c++) A[c] = add_rn(mul_rn(km, tm[c]), mul_rn(ko, to[c]));
    const T A2 = A[0] * A[0] + A[1] * A[1] + A[2] * A[2];
    T Amag, iA;
    if constexpr (sizeof(T) == 8) {
        if (!(A2 > T(0))) return out;
        Amag = sqrt_inv(A2, iA);
    } else {
        Amag = tsqrt(A2);
        if (!(Amag > T(0))) return out;
        iA = T(1) / Amag;
    }
    const T nh[3] = {A[0] * iA, A[1] * iA, A[2] * iA};

    // midpoint reconstruction of rho, vx, vy, vz, P on each side
    const int slot[5] = {R_RHO, R_V0, R_V0 + 1, R_V0 + 2, R_P};
    const T sm = mL ? T(0.5) : T(-0.5);
    T qL[5], qR[5];
#pragma unroll
    for (int f = 0; f < 5; f++) {
        const T* gm = m + R_G + 3 * f;
        const T* go = o + R_G + 3 * f;
        T qm = m[slot[f]] + sm * (gm[0] * d[0] + gm[1] * d[1] + gm[2] * d[2]);
        T qo = o[slot[f]] + (-sm) * (go[0] * d[0] + go[1] * d[1] + go[2] * d[2]);
        if (LIM) {
            qm = pair_limit<T>(qm, m[slot[f]], o[slot[f]]);
            qo = pair_limit<T>(qo, o[slot[f]], m[slot[f]]);
        }
        qL[f] = mL ? qm : qo;
        qR[f] = mL ? qo : qm;
    }
    const bool first = !(qL[0] > T(0)) || !(qL[4] > T(0)) || !(qR[0] > T(0)) || !(qR[4] > T(0));
    if (first) {
#pragma unroll
        for (int f = 0; f < 5; f++) {
            qL[f] = mL ? m[slot[f]] : o[slot[f]];
            qR[f] = mL ? o[slot[f]] : m[slot[f]];
        }
        out.fallback = 1;
    }
    // pressure difference across the face, P_R - P_L.  With FP32 records the
    // centre pressures' difference is taken in FP64 first (each record carries
    // its pressure in FP64): in dense, slow gas that difference is a small part
    // of P, and rounding each face pressure to FP32 would swamp it (and with it
    // the contact speed S*); the FP32 reconstruction offsets are added after.
    T dPRL;
    if constexpr (sizeof(T) == 8) {
        dPRL = qR[4] - qL[4];
    } else {
        const double Pm = __longlong_as_double(((long long)__float_as_int(m[1]) << 32) |
                                               (unsigned)__float_as_int(m[0]));
        const double Po = __longlong_as_double(((long long)__float_as_int(o[1]) << 32) |
                                               (unsigned)__float_as_int(o[0]));
        const double dc = mL ? Po - Pm : Pm - Po;
        // the offsets as the reconstruction formed them: (face - centre) per side
        const T offL = first ? T(0) : qL[4] - (mL ? m[R_P] : o[R_P]);
        const T offR = first ? T(0) : qR[4] - (mL ? o[R_P] : m[R_P]);
        dPRL = (T)dc + (offR - offL);
    }
    // face frame: the mean of the two particle velocities (commutative)
    const T w[3] = {T(0.5) * (m[R_V0] + o[R_V0]), T(0.5) * (m[R_V0 + 1] + o[R_V0 + 1]),
                    T(0.5) * (m[R_V0 + 2] + o[R_V0 + 2])};
    const T uL = (qL[1] - w[0]) * nh[0] + (qL[2] - w[1]) * nh[1] + (qL[3] - w[2]) * nh[2];
    const T uR = (qR[1] - w[0]) * nh[0] + (qR[2] - w[1]) * nh[1] + (qR[3] - w[2]) * nh[2];
    const T rL = qL[0], pL = qL[4], rR = qR[0], pR = qR[4];
    T cL, cR;
    sound_speeds(gamma * pL, rL, gamma * pR, rR, cL, cR);
    const T SL = (uL - cL < uR - cR) ? uL - cL : uR - cR;
    const T SR = (uL + cL > uR + cR) ? uL + cL : uR + cR;
    const T mLf = rL * (SL - uL), mRf = rR * (SR - uR);
    const T Ss = (dPRL + mLf * uL - mRf * uR) / (mLf - mRf);
    if (MFV) {
        mfv_flux<T>(qL, qR, w, nh, uL, uR, SL, SR, Ss, gamma, Amag, out);
        return out;
    }
    T Ps = T(0.5) * (pL + pR + mLf * (Ss - uL) + mRf * (Ss - uR));
    if (Ps < T(0)) {
        Ps = T(0);
        out.clamp = 1;
    }
    const T wn = w[0] * nh[0] + w[1] * nh[1] + w[2] * nh[2];
#pragma unroll
    for (int c = 0; c < 3; c++) out.Fp[c] = Ps * A[c];
    out.FE = Ps * (Ss + wn) * Amag;
    return out;
}

template <typename T>
__device__ __forceinline__ void load_rec(const T* __restrict__ rec, long long i, T v[32]);
template <>
__device__ __forceinline__ void load_rec<double>(const double* __restrict__ rec, long long i, double v[32]) {
    const double2* p = (const double2*)(rec + i * 32);
#pragma unroll
    for (int k = 0; k < 16; k++) {
        double2 t = p[k];
        v[2 * k] = t.x;
        v[2 * k + 1] = t.y;
    }
}
template <>
__device__ __forceinline__ void load_rec<float>(const float* __restrict__ rec, long long i, float v[32]) {
    const float4* p = (const float4*)(rec + i * 32);
#pragma unroll
    for (int k = 0; k < 8; k++) {
        float4 t = p[k];
        v[4 * k] = t.x;
        v[4 * k + 1] = t.y;
        v[4 * k + 2] = t.z;
        v[4 * k + 3] = t.w;
    }
}

// Hierarchical steps (the levelled pass): a pair {i, j} has level max(bin_i,
// bin_j); only pairs of level >= lmin are evaluated, and each particle's sums
// per level go to lev[(l * 4 + c) * n + i] (c: dp x, y, z, dE) for the levels
// >= lmin, the others keeping their values.  The sums of levels bin_i ..
// bin_i + kLevWin - 1 (a particle's pairs are never coarser than its own bin)
// are kept in registers; finer levels are summed in place in lev.
constexpr int kLevWin = 4;
struct Levels {
    const long long* bin;
    int lmin, nlev;
    double* lev;
    const long long* home;   // column of lev per particle (null: the particle's index)
};

// LDS of one wave's record gathers: the FP64 record (256 B), or the FP32 record
// (128 B) and the FP64 position from the packed neighbour record
template <typename T>
struct FluxLds;
template <>
struct FluxLds<double> {
    TeamLds<16> rec;
};
template <>
struct FluxLds<float> {
    TeamLds<8> rec;
    TeamLds<2> pos;
};

template <typename T, bool MFV, bool LIM, int SPLIT, bool LEV = false>
__device__ __forceinline__ void fluxes_body(const PassArrays& a, const Phys& ph, const int* __restrict__ counts,
                                            const int* __restrict__ list, const T* __restrict__ rec,
                                            const double4* __restrict__ prim, Counters* cnt,
                                            Levels lv = Levels{nullptr, 0, 0, nullptr, nullptr}) {
    cnt = counter_copy(cnt);
    __shared__ FluxLds<T> S;
    static_assert(!LEV || SPLIT == 1, "the levelled sums are one lane's");
    constexpr int kOwn = kWave / SPLIT;   // particles of the wave
    const int lane = threadIdx.x, sub = lane / kOwn;
    const int i = xcd_block() * kOwn + lane % kOwn;
    const bool act = i < a.n;
    const long long n = a.n;
    const int self = act ? i : a.n - 1;   // a record to load where a lane has no pair
    unsigned long long nfall = 0, nclamp = 0, nonfin = 0;
    const int cnum = act ? counts[i] : 0;
    T ri[32];
    // in the levelled pass most particles of a partial boundary have no
    // list: their record is not read (its values only enter pairs)
    if (cnum == 0 && (LEV || !act)) {
#pragma unroll
        for (int q = 0; q < 32; q++) ri[q] = T(0);
    } else {
        load_rec<T>(rec, i, ri);
    }
    double xi[3] = {0.0, 0.0, 0.0};
    if (act) {
        xi[0] = a.x[i];
        xi[1] = a.y[i];
        xi[2] = a.z[i];
    }
    const double vi[3] = {(double)ri[R_V0], (double)ri[R_V0 + 1], (double)ri[R_V0 + 2]};
    const double ci = (double)ri[R_C];
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    double accm = 0.0;
    double vs = 0.0;
    const T gam = (T)ph.gamma;
    int bi = 0;
    long long li = i;
    double lacc[kLevWin][4];
    if (LEV) {
        if (act) {
            bi = (int)lv.bin[i];
            if (lv.home) li = lv.home[i];
        }
#pragma unroll
        for (int w = 0; w < kLevWin; w++)
#pragma unroll
            for (int c = 0; c < 4; c++) lacc[w][c] = 0.0;
        if (act)
            for (int l = max(lv.lmin, bi + kLevWin); l < lv.nlev; l++)
                for (int c = 0; c < 4; c++) lv.lev[((long long)l * 4 + c) * n + li] = 0.0;
    }
    // One pair per lane and step, the wave running as far as its longest list:
    // while a pair is evaluated the next one's record is on its way to LDS, and
    // the index of the one after to a register.  A pair that is not due in the
    // levelled pass costs its bin alone (no flux, no signal speed: the last
    // boundary of a system step has every pair due, so the signal speeds it
    // leaves are complete), and a step without a due pair loads no records.
    const int kmax = __builtin_amdgcn_readfirstlane(wave_max_i((cnum + SPLIT - 1) / SPLIT));
    auto entry = [&](int k) {
        const int e = k * SPLIT + sub;
        return e < cnum ? list[(long long)e * n + i] : -1;
    };
    auto level = [&](int j) { return j >= 0 ? max(bi, (int)lv.bin[j]) : -1; };
    auto is_due = [&](int j, int l) { return j >= 0 && (!LEV || l >= lv.lmin); };
    auto start = [&](bool on, int j) {
        if (LEV && !__ballot(on)) return;
        const int jr = on ? j : self;
        team_load<32 * sizeof(T), 2 * sizeof(T)>(S.rec, rec, a.n, jr, lane);
        if constexpr (sizeof(T) == 4) team_load<128, 2>(S.pos, prim, a.n, jr, lane);
    };
    int j = entry(0), jn = entry(1);
    int lj = LEV ? level(j) : 0;
    bool due = is_due(j, lj);
    if (kmax > 0) start(due, j);
    for (int k = 0; k < kmax; k++) {
        T rj[32];
        double xj[3];
        wait_vmem();
        wave_lds_sync();
#pragma unroll
        for (int c = 0; c < (int)sizeof(T) * 2; c++) {
            const uint4 u = team_chunk(S.rec, c, lane);
            __builtin_memcpy(rj + c * (16 / sizeof(T)), &u, 16);
        }
        if constexpr (sizeof(T) == 8) {
            xj[0] = (double)rj[0];
            xj[1] = (double)rj[1];
            xj[2] = (double)rj[2];
        } else {
            const uint4 u = team_chunk(S.pos, 0, lane), v = team_chunk(S.pos, 1, lane);
            __builtin_memcpy(xj, &u, 16);
            __builtin_memcpy(xj + 2, &v, 8);
        }
        const int jc = j, lc = lj;
        const bool on = due;
        j = jn;
        lj = LEV ? level(j) : 0;
        due = is_due(j, lj);
        wave_lds_sync();
        wait_lds();
        if (k + 1 < kmax) start(due, j);
        jn = entry(k + 2);
        if (!on) continue;
        double dij[3];
        displacement(ph, xi, xj[0], xj[1], xj[2], dij);   // x_j - x_i
        const double r2 = dij[0] * dij[0] + dij[1] * dij[1] + dij[2] * dij[2];
        double r, ir;
        if constexpr (sizeof(T) == 8)
            r = sqrt_inv(r2, ir);
        else
            r = sqrt(r2);
        const bool iL = i < jc;
        // signal speed over the flux neighbours (the due ones in the levelled pass)
        auto signal = [&]() {
            const double cj = (double)rj[R_C];
            const double vd = (vi[0] - (double)rj[R_V0]) * dij[0] + (vi[1] - (double)rj[R_V0 + 1]) * dij[1] +
                              (vi[2] - (double)rj[R_V0 + 2]) * dij[2];
            const double proj = sizeof(T) == 8 ? -vd * ir : -vd / r;
            vs = fmax(vs, ci + cj - fmin(proj, 0.0));
        };
        // canonical displacement x_R - x_L: the minimum image commutes with
        // negation exactly, so both owners of the pair hold the same bits
        const double sg = iL ? 1.0 : -1.0;
        const T dT[3] = {(T)(sg * dij[0]), (T)(sg * dij[1]), (T)(sg * dij[2])};
        PairOut<T> o = pair_flux<T, MFV, LIM>(ri, rj, iL, dT, (T)r, gam);
        const double s = iL ? 1.0 : -1.0;
        if (MFV) accm -= s * (double)o.Fm;
        acc[0] -= s * (double)o.Fp[0];
        acc[1] -= s * (double)o.Fp[1];
        acc[2] -= s * (double)o.Fp[2];
        acc[3] -= s * (double)o.FE;
        nfall += o.fallback;
        nclamp += o.clamp;
        signal();
        if (LEV) {
            const double F[4] = {(double)o.Fp[0], (double)o.Fp[1], (double)o.Fp[2], (double)o.FE};
            const int w = lc - bi;
            if (w == 0) {   // both particles in one bin: most pairs
#pragma unroll
                for (int c = 0; c < 4; c++) lacc[0][c] = lacc[0][c] - s * F[c];
            } else if (w < kLevWin) {
#pragma unroll
                for (int q = 1; q < kLevWin; q++)
#pragma unroll
                    for (int c = 0; c < 4; c++) lacc[q][c] = (q == w) ? lacc[q][c] - s * F[c] : lacc[q][c];
            } else {
                for (int c = 0; c < 4; c++) lv.lev[((long long)lc * 4 + c) * n + li] -= s * F[c];
            }
        }
    }
#pragma unroll
    for (int c = 0; c < 4; c++) split_sum<SPLIT>(acc[c]);
    if (MFV) split_sum<SPLIT>(accm);
    split_max<SPLIT>(vs);
    if (act && sub == 0) {
        if (LEV) {
#pragma unroll
            for (int w = 0; w < kLevWin; w++) {
                const int l = bi + w;
                if (l >= lv.lmin && l < lv.nlev)
#pragma unroll
                    for (int c = 0; c < 4; c++) lv.lev[((long long)l * 4 + c) * n + li] = lacc[w][c];
            }
            // due levels coarser than the particle's own bin hold no pair of it
            for (int l = lv.lmin; l < min(bi, lv.nlev); l++)
                for (int c = 0; c < 4; c++) lv.lev[((long long)l * 4 + c) * n + li] = 0.0;
        }
        a.dp[i] = acc[0];
        a.dp[n + i] = acc[1];
        a.dp[2 * n + i] = acc[2];
        a.dE[i] = acc[3];
        a.vsig[i] = vs;
        if (MFV) a.dm[i] = accm;
        if (!isfinite(acc[0]) || !isfinite(acc[1]) || !isfinite(acc[2]) || !isfinite(acc[3]) || !isfinite(accm)) {
            nonfin = 1;
            flag_index(cnt, i);
        }
    }
    count_add(&cnt->fallbacks, nfall);
    count_add(&cnt->clamps, nclamp);
    count_add(&cnt->nonfinite, nonfin);
}

// One kernel per record precision: each pair holds both records in registers.
// The neighbours' records come by lane teams (team_load): per pair the FP64 form
// made 16 loads of 64 cache lines each and the FP32 form 11, which the L1 takes
// at about one line a clock and compute unit, the whole of the kernels' time on
// even sets.  Now the arithmetic of the longest list of a wave bounds them.
// Blocks of one wave: a block's LDS (16.3 KB FP64, 10.5 KB FP32) is free again
// as soon as its wave ends.  The FP64 form runs at two waves per SIMD (its two
// records alone are 128 VGPRs), the FP32 form at three.  Measured: FP64 MFM,
// lattice 2.1M 1.84 -> 1.2 ms, clustered 16.8M 19.4 -> 14.0 ms (15.7 before the
// 32-bit record offsets and the square roots with their reciprocals); mixed MFM,
// shock tube 295k 0.232 -> 0.181 ms; limited FP64, clustered 2.1M 4.35 -> 3.47
// ms; levelled, hierarchical step of 2.1M 0.89 -> 0.69 ms a launch.
// A particle's list is shared by SPLIT lanes: eight up to kFluxSplit8 particles
// (too few waves for the chip otherwise), two beyond (a wave of 32 particles
// waits for the longest of 32 lists, not of 64); the levelled form keeps one.
// Measured, one / two / four / eight lanes: lattice 4,096 52 / 29 / 18 / 13 us,
// 32,768 54 / 34 / 30 / 33, 64,000 59 / 48 / 49 / 54, 2.1M 1.10 / 1.09 / 1.14 ms;
// clustered 32,768 201 / 107 / 63 / 52 us, 64,000 329 / 168 / 104 / 80, 16.8M
// 13.9 / 12.6 / 12.2 ms; mixed, shock tube 295k 0.189 / 0.145 / 0.141 ms.
constexpr int kFluxSplit8 = 49152;
constexpr int kFlux64Waves = 2;
constexpr int kFluxMfvWaves = kFlux64Waves;
template <bool LIM, int SPLIT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kFlux64Waves))) void k_fluxes_f64(PassArrays a, Phys ph, const int* __restrict__ counts,
                                                    const int* __restrict__ list, const double* __restrict__ rec,
                                                    const double4* __restrict__ prim, Counters* cnt) {
    fluxes_body<double, false, LIM, SPLIT>(a, ph, counts, list, rec, prim, cnt);
}

// The levelled pass of hierarchical steps (MFM, FP64 records).
template <bool LIM>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kFlux64Waves))) void k_fluxes_levels(
    PassArrays a, Phys ph, const int* __restrict__ counts, const int* __restrict__ list,
    const double* __restrict__ rec, const double4* __restrict__ prim, Counters* cnt, Levels lv) {
    fluxes_body<double, false, LIM, 1, true>(a, ph, counts, list, rec, prim, cnt, lv);
}

// The finite-volume form, FP64 records only, at two waves per SIMD like the
// FP64 form (at three its extra live values spill).
template <bool LIM, int SPLIT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kFluxMfvWaves))) void k_fluxes_mfv(PassArrays a, Phys ph, const int* __restrict__ counts,
                                                    const int* __restrict__ list, const double* __restrict__ rec,
                                                    const double4* __restrict__ prim, Counters* cnt) {
    fluxes_body<double, true, LIM, SPLIT>(a, ph, counts, list, rec, prim, cnt);
}

constexpr int kFlux32Waves = 3;
template <bool LIM, int SPLIT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kFlux32Waves)))
void k_fluxes_f32(PassArrays a, Phys ph, const int* __restrict__ counts, const int* __restrict__ list,
                  const float* __restrict__ rec, const double4* __restrict__ prim, Counters* cnt) {
    fluxes_body<float, false, LIM, SPLIT>(a, ph, counts, list, rec, prim, cnt);
}

// The finite-volume form on the FP32 records of the mixed form.
template <bool LIM, int SPLIT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kFlux32Waves)))
void k_fluxes_mfv_f32(PassArrays a, Phys ph, const int* __restrict__ counts, const int* __restrict__ list,
                      const float* __restrict__ rec, const double4* __restrict__ prim, Counters* cnt) {
    fluxes_body<float, true, LIM, SPLIT>(a, ph, counts, list, rec, prim, cnt);
}

// ------------------------------------------------------------------ launchers
static int blocks_of(int n, int b) { return (n + b - 1) / b; }
constexpr int kFallbackWaves = 1024;

void launch_solve_h(const PassArrays& a, const TreeDesc& td, const int2* tab,
                    const double4* pos, const unsigned long long* keys, const Phys& ph, Counters* cnt, double* rl, int* list,
                    int* gcount,
                    int* counts, int* fb_list, unsigned long long* fb_count, int* fb2_list,
                    unsigned long long* fb2_count, hipEvent_t t0, hipEvent_t t1, hipStream_t s) {
    const bool direct = a.n <= kDirectMax;
    if (!direct) {
        launch_fill_u64(1, fb_count, 0ull, s);
        launch_fill_u64(1, fb2_count, 0ull, s);
    }
    if (t0) hipEventRecord(t0, s);
    if (direct) {
        k_solve_start<false><<<blocks_of(a.n, 256), 256, 0, s>>>(a, td, tab, keys, ph, rl, fb_list, fb_count, fb2_count,
                                                                 nullptr);
    } else {
        k_solve_h<false><<<blocks_of(a.n, 256), 256, 0, s>>>(a, td, tab, pos, keys, ph, cnt, rl, list, gcount, counts,
                                                             fb_list, fb_count, nullptr, nullptr);
        k_root_h<false><<<blocks_of(a.n, 256), 256, 0, s>>>(a, ph.n_ngb, ph.h_maxit, cnt, rl, list, gcount, counts,
                                                            fb_list, fb_count, nullptr);
    }
    // one wave per handed-over particle, striding over the count left on the device
    k_solve_h_wave<<<std::min(a.n, kWaveBlocks), 64, 0, s>>>(a, td, tab, pos, ph, cnt, fb_list, fb_count, rl, list,
                                                             gcount, counts, fb2_list, fb2_count, nullptr, !direct);
    k_solve_h_fallback<<<std::min(a.n, kFallbackWaves), 64, 0, s>>>(a, td, tab, pos, ph, cnt, fb2_list, fb2_count, list,
                                                                    gcount, counts, nullptr);
    if (t1) hipEventRecord(t1, s);
}

template <int SPLIT>
static void launch_gradients_split(const PassArrays& a, const Phys& ph, const int* gcount, int* counts, int* list,
                                   const Bins& bins, int mixed, double4* prim, void* rec, Counters* cnt, hipStream_t s) {
    const int blocks = blocks_of(a.n, kWave / SPLIT);
    if (mixed)
        k_gradients<true, false, SPLIT><<<blocks, kWave, 0, s>>>(a, ph, gcount, counts, list, bins, prim, rec, cnt,
                                                                 nullptr, nullptr);
    else
        k_gradients<false, false, SPLIT><<<blocks, kWave, 0, s>>>(a, ph, gcount, counts, list, bins, prim, rec, cnt,
                                                                  nullptr, nullptr);
}

void launch_gradients(const PassArrays& a, const Phys& ph, const int* gcount, int* counts, int* list, int2* bin_entry, int* bin_fill,
                      int mixed, double4* prim, void* rec, Counters* cnt, hipEvent_t t0, hipEvent_t t1,
                      hipStream_t s) {
    const Bins bins{bin_entry, bin_fill};
    k_pack_prim<<<blocks_of(a.n, 256), 256, 0, s>>>(a, ph, prim, bin_fill);
    if (t0) hipEventRecord(t0, s);
    if (a.n <= kGradSplit4)
        launch_gradients_split<4>(a, ph, gcount, counts, list, bins, mixed, prim, rec, cnt, s);
    else if (a.n <= kGradSplit2)
        launch_gradients_split<2>(a, ph, gcount, counts, list, bins, mixed, prim, rec, cnt, s);
    else
        launch_gradients_split<1>(a, ph, gcount, counts, list, bins, mixed, prim, rec, cnt, s);
    if (t1) hipEventRecord(t1, s);
    k_sort_tails<<<blocks_of(a.n, 256), 256, 0, s>>>(a.n, ph.max_ngb, gcount, counts, list, bins, cnt);
}

void launch_solve_h_active(const PassArrays& a, const TreeDesc& td, const int2* tab, const double4* pos,
                           const unsigned long long* keys, const Phys& ph, Counters* cnt, const unsigned char* mode, const double* pad, double* rl,
                           int* list, int* gcount, int* counts, int* fb_list, unsigned long long* fb_count,
                           int* fb2_list, unsigned long long* fb2_count, hipStream_t s) {
    launch_fill_u64(1, fb_count, 0ull, s);
    launch_fill_u64(1, fb2_count, 0ull, s);
    const bool direct = a.n <= kDirectMax;
    if (direct) {
        k_solve_start<true><<<blocks_of(a.n, 256), 256, 0, s>>>(a, td, tab, keys, ph, rl, fb_list, fb_count, fb2_count,
                                                                mode);
    } else {
        k_solve_h<true><<<blocks_of(a.n, 256), 256, 0, s>>>(a, td, tab, pos, keys, ph, cnt, rl, list, gcount, counts,
                                                            fb_list, fb_count, mode, pad);
        k_root_h<true><<<blocks_of(a.n, 256), 256, 0, s>>>(a, ph.n_ngb, ph.h_maxit, cnt, rl, list, gcount, counts,
                                                           fb_list, fb_count, mode);
    }
    k_solve_h_wave<<<std::min(a.n, kWaveBlocks), 64, 0, s>>>(a, td, tab, pos, ph, cnt, fb_list, fb_count, rl, list,
                                                             gcount, counts, fb2_list, fb2_count, pad, !direct);
    k_solve_h_fallback<<<std::min(a.n, kFallbackWaves), 64, 0, s>>>(a, td, tab, pos, ph, cnt, fb2_list, fb2_count, list,
                                                                    gcount, counts, pad);
    k_gather_kept<<<blocks_of(a.n, 256), 256, 0, s>>>(a, td, tab, pos, ph, mode, pad, list, gcount, counts);
}

void launch_gradients_active(const PassArrays& a, const Phys& ph, const unsigned char* mode, const long long* home,
                             const int* gcount, int* counts, int* list, int2* bin_entry, int* bin_fill, double4* prim, void* rec,
                             Counters* cnt, hipStream_t s) {
    const Bins bins{bin_entry, bin_fill};
    k_pack_prim_active<<<blocks_of(a.n, 256), 256, 0, s>>>(a, ph, gcount, mode, list, prim, bin_fill);
    k_gradients<false, true, 1><<<blocks_of(a.n, kWave), kWave, 0, s>>>(a, ph, gcount, counts, list, bins, prim, rec, cnt,
                                                                 mode, home);
    k_sort_tails<<<blocks_of(a.n, 256), 256, 0, s>>>(a.n, ph.max_ngb, gcount, counts, list, bins, cnt);
    k_pack_rec_kept<<<blocks_of(a.n, 256), 256, 0, s>>>(a, ph, mode, home, counts, (double*)rec);
}

template <bool LIM, int SPLIT>
static void launch_fluxes_split(const PassArrays& a, const Phys& ph, const int* counts, const int* list, int mixed,
                                int mfv, const void* rec, const double4* prim, Counters* cnt, hipStream_t s) {
    const int blocks = blocks_of(a.n, kWave / SPLIT);
    if (mfv && mixed)
        k_fluxes_mfv_f32<LIM, SPLIT><<<blocks, kWave, 0, s>>>(a, ph, counts, list, (const float*)rec, prim, cnt);
    else if (mfv)
        k_fluxes_mfv<LIM, SPLIT><<<blocks, kWave, 0, s>>>(a, ph, counts, list, (const double*)rec, prim, cnt);
    else if (mixed)
        k_fluxes_f32<LIM, SPLIT><<<blocks, kWave, 0, s>>>(a, ph, counts, list, (const float*)rec, prim, cnt);
    else
        k_fluxes_f64<LIM, SPLIT><<<blocks, kWave, 0, s>>>(a, ph, counts, list, (const double*)rec, prim, cnt);
}

template <bool LIM>
static void launch_fluxes_lim(const PassArrays& a, const Phys& ph, const int* counts, const int* list, int mixed,
                              int mfv, const void* rec, const double4* prim, Counters* cnt, hipStream_t s) {
    if (a.n <= kFluxSplit8)
        launch_fluxes_split<LIM, 8>(a, ph, counts, list, mixed, mfv, rec, prim, cnt, s);
    else
        launch_fluxes_split<LIM, 2>(a, ph, counts, list, mixed, mfv, rec, prim, cnt, s);
}

void launch_fluxes_levels(const PassArrays& a, const Phys& ph, const int* counts, const int* list, const void* rec,
                          const double4* prim, Counters* cnt, const long long* bin, int lmin, int nlev, double* lev,
                          const long long* home, hipStream_t s) {
    const Levels lv{bin, lmin, nlev, lev, home};
    if (ph.limiter)
        k_fluxes_levels<true><<<blocks_of(a.n, kWave), kWave, 0, s>>>(a, ph, counts, list, (const double*)rec, prim, cnt, lv);
    else
        k_fluxes_levels<false><<<blocks_of(a.n, kWave), kWave, 0, s>>>(a, ph, counts, list, (const double*)rec, prim, cnt, lv);
}

void launch_fluxes(const PassArrays& a, const Phys& ph, const int* counts, const int* list, int mixed, int mfv,
                   const void* rec, const double4* prim, Counters* cnt, hipStream_t s) {
    if (ph.limiter)
        launch_fluxes_lim<true>(a, ph, counts, list, mixed, mfv, rec, prim, cnt, s);
    else
        launch_fluxes_lim<false>(a, ph, counts, list, mixed, mfv, rec, prim, cnt, s);
}

}  // namespace mfm
