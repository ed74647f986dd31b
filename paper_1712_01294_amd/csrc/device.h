// Device-side building blocks of the gfx950 MFM pass: cubic-spline kernel,
// minimum-image displacement, and the wave-cooperative scans over the cell
// tables that the Morton-sorted particle order defines (one (start, end)
// range per cell of every level of an implicit octree).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mfm {

constexpr int kMaxLevels = 12;   // levels 0..kMaxLevels-1
constexpr int kWave = 64;

// Everything a kernel needs to walk the cell tables, passed by value.
struct TreeDesc {
    int bmax;                        // deepest level
    int ktot;                        // key bits at bmax
    int actmask[kMaxLevels];         // bit d set when axis d refines at level l
    int kbits[kMaxLevels];           // key-prefix bits of a level-l cell
    long long tab_off[kMaxLevels];   // offset of level l in the (start, end) table
    double cs[kMaxLevels][3];        // cell side per axis at level l
    int ncell[kMaxLevels][3];        // cells per axis at level l (a power of two)
    unsigned long long mask[kMaxLevels][3];  // key-prefix bits of axis d at level l
    double box[3];
    int periodic[3];
    int qbits[3];                    // quantisation bits per axis
};

// Run-time physics parameters shared by the pass kernels.
struct Phys {
    double gamma;
    double n_ngb;
    double beta;
    double cond_max;
    double box[3];
    int periodic[3];
    int h_maxit;
    int max_ngb;
    int limiter;          // 1: pairwise face limiter and condition-adaptive beta
    double beta_min, cond_lo, cond_hi;
};

// Device counters (all updated with atomics, read by the host after a sync).
// There are kCounterCopies copies, kCounterStride bytes apart; a block updates
// the copy of its blockIdx modulo the count, which spreads the atomics of a
// launch over as many cache lines (all on one line serialise in one L2
// channel), and the host combines the copies when it reads them.
struct Counters {
    unsigned long long list_entries;
    unsigned long long list_max;
    unsigned long long h_iters;
    unsigned long long h_iters_max;
    unsigned long long noconv;
    unsigned long long minimage;
    unsigned long long overflow;
    unsigned long long illcond;
    unsigned long long fallbacks;
    unsigned long long clamps;
    unsigned long long nonfinite;
    unsigned long long floors;
    unsigned long long first_bad;    // min index (init ~0ull)
    unsigned long long cond_bits;    // max of the positive double cond, as bits
    unsigned long long h_rounds_max; // most group scans a kernel-length solve needed
    unsigned long long h_fallback;   // particles solved by the per-particle kernel
    unsigned long long h_rounds3;    // particles that needed three or more scans
    unsigned long long gather_entries;  // sum of the gather-list lengths
    unsigned long long h_rescan;     // particles the rescanning kernel-length solver took
};
constexpr int kCounterCopies = 32;
constexpr int kCounterStride = 256;
static_assert(sizeof(Counters) <= kCounterStride, "counter copies overlap");

// the copy of the counters the calling block updates
__device__ __forceinline__ Counters* counter_copy(Counters* base) {
    return (Counters*)((char*)base + (blockIdx.x & (kCounterCopies - 1)) * kCounterStride);
}

// sqrt(x) for 0 <= x far from the ends of the exponent range (a squared
// distance): the steps of the correctly rounded sqrt without its rescaling of
// arguments below 2^-767
__device__ __forceinline__ double sqrt_mid(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    g = fma(fma(-g, g, x), h, g);
    g = fma(fma(-g, g, x), h, g);
    return x > 0.0 ? g : 0.0;
}

// 2^-700 <= x < 2^700
__device__ __forceinline__ bool is_mid(double x) {
    return (unsigned)__double2hiint(x) - (323u << 20) < (1400u << 20);
}

// sqrt(x) and 1/sqrt(x) together for x as in is_mid (the correctly rounded
// sqrt's steps, its half reciprocal refined once more: 12 instructions against 33
// of a square root and a division; the reciprocal is within 1.5 ulp)
__device__ __forceinline__ double sqrt_inv_mid(double x, double& inv) {
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    g = fma(fma(-g, g, x), h, g);
    const double e = fma(-h, g, 0.5);
    g = fma(fma(-g, g, x), h, g);
    inv = 2.0 * fma(h, e, h);
    return g;
}

// the same for every x
__device__ __forceinline__ double sqrt_inv(double x, double& inv) {
    if (__builtin_expect(is_mid(x), 1)) return sqrt_inv_mid(x, inv);
    const double g = sqrt(x);
    inv = 1.0 / g;
    return g;
}

// ---------------------------------------------------------------- kernel
// Cubic spline with support radius H: W = 8/(pi H^3) w(q), q = r/H,
// w = 1 - 6q^2 + 6q^3 (q <= 1/2), 2(1-q)^3 (1/2 < q <= 1), 0 beyond.
// With t = max(1 - q, 0) and u = max(1/2 - q, 0) both pieces are one
// expression, w = 2 t^3 - 8 u^3 (expanding 2(1-q)^3 - (1-2q)^3 gives the inner
// piece), and q w'(q) = q (24 u^2 - 6 t^2): no selects or branches, so lanes
// with q on different pieces run the same instructions.
__device__ __forceinline__ double spline_pos(double a) { return fmax(a, 0.0); }
__device__ __forceinline__ float spline_pos(float a) { return fmaxf(a, 0.0f); }

template <typename T>
__device__ __forceinline__ T spline_w(T q) {
    const T t = spline_pos(T(1) - q);
    const T u = spline_pos(T(0.5) - q);
    return T(2) * (t * t) * t - T(8) * (u * u) * u;
}

// dw/dq
template <typename T>
__device__ __forceinline__ T spline_dw(T q) {
    const T t = spline_pos(T(1) - q);
    const T u = spline_pos(T(0.5) - q);
    return T(24) * (u * u) - T(6) * (t * t);
}

// q * dw/dq
template <typename T>
__device__ __forceinline__ T spline_qdw(T q) {
    const T t = spline_pos(T(1) - q);
    const T u = spline_pos(T(0.5) - q);
    return q * (T(24) * (u * u) - T(6) * (t * t));
}

template <typename T>
__device__ __forceinline__ T kernel_norm(T H) {
    return T(2.5464790894703255) / (H * H * H);  // 8/pi / H^3
}

// x_j - x_i on one axis, moved to the nearest periodic image
__device__ __forceinline__ double min_image(double d, double L, int periodic) {
    if (periodic) {
        if (d > 0.5 * L) d -= L;
        else if (d < -0.5 * L) d += L;
    }
    return d;
}

// ------------------------------------------------------------ wave collectives
// All 64 lanes participate.  Exchanges go through lane permutes of the vector
// ALU (halves, rows of 16, rotations within a row, quads), not through LDS: six
// dependent LDS permutes per 32 bits cost a reduction some 600 cycles, and a
// scan pass takes eight reductions and a prefix sum per 64 cells.  The pairing
// is that of a butterfly over distances 32, 16, 8, 4, 2, 1 (after the step over
// 8 a row's lanes hold equal values 8 apart, so a rotation by 4 gives the value
// of the lane 4 across), so sums take the same order on every lane.
__device__ __forceinline__ void swap_halves(unsigned& a, unsigned& b) {   // upper half of a <-> lower half of b
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}
__device__ __forceinline__ void swap_rows(unsigned& a, unsigned& b) {     // odd rows of a <-> even rows of b
    const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}
template <int CTRL>
__device__ __forceinline__ unsigned lane_move(unsigned v) {
    return (unsigned)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xf, 0xf, true);
}

template <typename T>
struct Words {
    static constexpr int n = sizeof(T) / 4;
    unsigned w[n];
    __device__ __forceinline__ static Words of(T v) { return __builtin_bit_cast(Words, v); }
    __device__ __forceinline__ T value() const { return __builtin_bit_cast(T, *this); }
};

template <typename T, typename Op>
__device__ __forceinline__ T wave_reduce(T v, Op op) {
    using W = Words<T>;
    W a = W::of(v), b = a;
#pragma unroll
    for (int k = 0; k < W::n; k++) swap_halves(a.w[k], b.w[k]);
    a = b = W::of(op(a.value(), b.value()));
#pragma unroll
    for (int k = 0; k < W::n; k++) swap_rows(a.w[k], b.w[k]);
    a = W::of(op(a.value(), b.value()));
#pragma unroll
    for (int k = 0; k < W::n; k++) b.w[k] = lane_move<0x128>(a.w[k]);   // row rotated by 8
    a = W::of(op(a.value(), b.value()));
#pragma unroll
    for (int k = 0; k < W::n; k++) b.w[k] = lane_move<0x124>(a.w[k]);   // by 4
    a = W::of(op(a.value(), b.value()));
#pragma unroll
    for (int k = 0; k < W::n; k++) b.w[k] = lane_move<0x4e>(a.w[k]);    // quad 2 3 0 1
    a = W::of(op(a.value(), b.value()));
#pragma unroll
    for (int k = 0; k < W::n; k++) b.w[k] = lane_move<0xb1>(a.w[k]);    // quad 1 0 3 2
    return op(a.value(), b.value());
}

// op over the SPLIT lanes that share a particle: lanes 64 / SPLIT apart (SPLIT
// 1, 2, 4 or 8), the same order on each
template <int SPLIT, typename T, typename Op>
__device__ __forceinline__ T split_reduce(T v, Op op) {
    using W = Words<T>;
    if constexpr (SPLIT >= 2) {
        W a = W::of(v), b = a;
#pragma unroll
        for (int k = 0; k < W::n; k++) swap_halves(a.w[k], b.w[k]);
        v = op(a.value(), b.value());
    }
    if constexpr (SPLIT >= 4) {
        W a = W::of(v), b = a;
#pragma unroll
        for (int k = 0; k < W::n; k++) swap_rows(a.w[k], b.w[k]);
        v = op(a.value(), b.value());
    }
    if constexpr (SPLIT >= 8) {
        W b = W::of(v);
#pragma unroll
        for (int k = 0; k < W::n; k++) b.w[k] = lane_move<0x128>(b.w[k]);   // row rotated by 8
        v = op(v, b.value());
    }
    return v;
}
template <int SPLIT>
__device__ __forceinline__ void split_sum(double& v) {
    v = split_reduce<SPLIT>(v, [](double a, double b) { return a + b; });
}
template <int SPLIT>
__device__ __forceinline__ void split_max(double& v) {
    v = split_reduce<SPLIT>(v, [](double a, double b) { return fmax(a, b); });
}
template <int SPLIT>
__device__ __forceinline__ void split_min(double& v) {
    v = split_reduce<SPLIT>(v, [](double a, double b) { return fmin(a, b); });
}

// the sums of u and v at once, each in the order of a sum of its own: after the
// first step the lower half of the wave carries u and the upper half v
__device__ __forceinline__ void wave_sum2_d(double u, double v, double& su, double& sv) {
    using W = Words<double>;
    W a = W::of(u), b = W::of(v);
#pragma unroll
    for (int k = 0; k < W::n; k++) swap_halves(a.w[k], b.w[k]);
    a = b = W::of(a.value() + b.value());
#pragma unroll
    for (int k = 0; k < W::n; k++) swap_rows(a.w[k], b.w[k]);
    a = W::of(a.value() + b.value());
#pragma unroll
    for (int k = 0; k < W::n; k++) b.w[k] = lane_move<0x128>(a.w[k]);
    a = W::of(a.value() + b.value());
#pragma unroll
    for (int k = 0; k < W::n; k++) b.w[k] = lane_move<0x124>(a.w[k]);
    a = W::of(a.value() + b.value());
#pragma unroll
    for (int k = 0; k < W::n; k++) b.w[k] = lane_move<0x4e>(a.w[k]);
    a = W::of(a.value() + b.value());
#pragma unroll
    for (int k = 0; k < W::n; k++) b.w[k] = lane_move<0xb1>(a.w[k]);
    a = W::of(a.value() + b.value());
    Words<double> lo, hi;
#pragma unroll
    for (int k = 0; k < W::n; k++) {
        lo.w[k] = (unsigned)__builtin_amdgcn_readlane((int)a.w[k], 0);
        hi.w[k] = (unsigned)__builtin_amdgcn_readlane((int)a.w[k], 32);
    }
    su = lo.value();
    sv = hi.value();
}

__device__ __forceinline__ double wave_sum_d(double v) {
    return wave_reduce(v, [](double a, double b) { return a + b; });
}
__device__ __forceinline__ double wave_min_d(double v) {
    return wave_reduce(v, [](double a, double b) { return fmin(a, b); });
}
__device__ __forceinline__ double wave_max_d(double v) {
    return wave_reduce(v, [](double a, double b) { return fmax(a, b); });
}
__device__ __forceinline__ int wave_min_i(int v) {
    return wave_reduce(v, [](int a, int b) { return min(a, b); });
}
__device__ __forceinline__ int wave_max_i(int v) {
    return wave_reduce(v, [](int a, int b) { return max(a, b); });
}

// inclusive prefix of op over the lanes, `none` its neutral value
template <typename Op>
__device__ __forceinline__ int wave_prefix(int v, int none, Op op) {
    v = op(v, __builtin_amdgcn_update_dpp(none, v, 0x111, 0xf, 0xf, false));   // from 1, 2, 4, 8 lanes below, in the row
    v = op(v, __builtin_amdgcn_update_dpp(none, v, 0x112, 0xf, 0xf, false));
    v = op(v, __builtin_amdgcn_update_dpp(none, v, 0x114, 0xf, 0xf, false));
    v = op(v, __builtin_amdgcn_update_dpp(none, v, 0x118, 0xf, 0xf, false));
    v = op(v, __builtin_amdgcn_update_dpp(none, v, 0x142, 0xa, 0xf, false));   // last lane of rows 0, 2 to rows 1, 3
    v = op(v, __builtin_amdgcn_update_dpp(none, v, 0x143, 0xc, 0xf, false));   // lane 31 to the upper half
    return v;
}
__device__ __forceinline__ int wave_prefix_sum(int v) {
    return wave_prefix(v, 0, [](int a, int b) { return a + b; });
}
__device__ __forceinline__ int wave_prefix_max(int v) {
    return wave_prefix(v, -1, [](int a, int b) { return max(a, b); });
}

// a value known to be equal on all lanes, moved to scalar registers
__device__ __forceinline__ double uniform_d(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readfirstlane((int)(b & 0xffffffffll));
    const int hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// order the LDS traffic of one wave (lanes read what other lanes wrote)
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ------------------------------------------------------- gathers by lane teams
// The first C 16-byte chunks of one record per lane, lane l's at base + STRIDE
// j(l), through LDS.  A load whose 64 lanes each read 16 bytes of a record of their own looks
// up 64 cache lines, and the L1 takes about one a clock: with 16 such loads per
// neighbour the FP64 flux kernel spent 1.77 ms of its 1.80 on the lookups
// (2.1M particles).  Here C neighbouring lanes read one record's chunks side by
// side, straight into LDS (64 / C records per load instruction), and each lane
// reads its record back from there.  Chunk c of lane r's record sits at
// position (c + r) mod C, so the lanes' reads of one chunk fall in different
// banks.  C is a power of two.
template <int C>
struct TeamLds {
    uint4 rec[kWave * C];
    int idx[kWave];
};

// LDS reads issued so far have returned / vector memory operations have completed
__device__ __forceinline__ void wait_lds() { __builtin_amdgcn_s_waitcnt(0xc07f); }
__device__ __forceinline__ void wait_vmem() { __builtin_amdgcn_s_waitcnt(0x0f70); }

// starts the loads of records j (one per lane, all 64 lanes) of the n records at
// base; the earlier records' reads must have returned.  Chunks from USED on are
// left out.  Up to 4 GiB of records are addressed by 32-bit offsets (one
// instruction a load instead of four).
template <int STRIDE, int USED, int C>
__device__ __forceinline__ void team_load(TeamLds<C>& S, const void* __restrict__ base, int n, int j, int lane) {
    typedef __attribute__((address_space(3))) uint4 LdsChunk;
    typedef __attribute__((address_space(1))) char Global;
    constexpr int kTeams = kWave / C;
    S.idx[(lane % kTeams) * C + lane / kTeams] = j;
    wave_lds_sync();
    const int team = lane / C, p = lane % C;
    int js[C];
#pragma unroll
    for (int q = 0; q < C; q++) js[q] = S.idx[team * C + q];
    wave_lds_sync();
    wait_lds();
    LdsChunk* to = (LdsChunk*)S.rec;
    const Global* from = (const Global*)base;
    if ((unsigned long long)n * STRIDE <= 1ull << 32) {
#pragma unroll
        for (int q = 0; q < C; q++) {
            const int c = (p - kTeams * q - team) & (C - 1);
            if (USED == C || c < USED)
                __builtin_amdgcn_global_load_lds(from + ((unsigned)js[q] * (unsigned)STRIDE + (unsigned)c * 16u),
                                                 to + q * kWave, 16, 0, 0);
        }
    } else {
#pragma unroll
        for (int q = 0; q < C; q++) {
            const int c = (p - kTeams * q - team) & (C - 1);
            if (USED == C || c < USED)
                __builtin_amdgcn_global_load_lds(from + ((size_t)(unsigned)js[q] * STRIDE + c * 16), to + q * kWave, 16,
                                                 0, 0);
        }
    }
}

// The other way: the lanes put the chunks of their records (team_put), then C
// neighbouring lanes store one record's chunks side by side, to base + STRIDE r
// for the lanes r whose bit is set in `lanes`.
template <int C>
__device__ __forceinline__ void team_put(TeamLds<C>& S, int c, int lane, const uint4& u) {
    S.rec[lane * C + ((c + lane) & (C - 1))] = u;
}
template <int STRIDE, int C>
__device__ __forceinline__ void team_store(const TeamLds<C>& S, void* __restrict__ base, unsigned long long lanes,
                                           int lane) {
    constexpr int kTeams = kWave / C;
    const int team = lane / C, p = lane % C;
#pragma unroll
    for (int q = 0; q < C; q++) {
        const int r = kTeams * q + team, c = (p - r) & (C - 1);
        if ((lanes >> r) & 1) *(uint4*)((char*)base + r * STRIDE + c * 16) = S.rec[q * kWave + lane];
    }
}

// chunk c of the lane's record, after wait_vmem
template <int C>
__device__ __forceinline__ uint4 team_chunk(const TeamLds<C>& S, int c, int lane) {
    return S.rec[lane * C + ((c + lane) & (C - 1))];
}

// ------------------------------------------------- wave-cooperative cell scan
// A group of lanes (Morton neighbours with similar trial radii) scans the union
// of their neighbourhoods together: the cells of one table level whose boxes
// come within Rq of the group's bounding box, on the finest level whose cells
// are at least kScanScale Rq wide.  Cells are taken 64 at a time, one per lane
// (key, table entry, periodic image); their particles are then staged 64 at a
// time in LDS with coalesced loads, already moved to the periodic image next to
// the group, and every lane tests each staged particle against its own sphere.
// The loop structure is the same for all lanes, so the wave never diverges on
// cell or particle counts and no lane waits on a dependent gather of its own.
// Cell keys come from per-axis cell coordinates deposited into the key bits of
// that axis (cells per axis are a power of two).
constexpr double kScanScale = 0.35;

// scatter the low bits of v into the set bits of mask (lowest first); bits of v
// beyond the mask's population are dropped, which reduces v modulo 2^popcount
__device__ __forceinline__ unsigned long long deposit_bits(unsigned v, unsigned long long mask) {
    unsigned long long r = 0;
    while (mask && v) {
        const unsigned long long low = mask & (~mask + 1);
        if (v & 1u) r |= low;
        v >>= 1;
        mask &= mask - 1;
    }
    return r;
}

// the low ten bits of v, two zero bits between neighbours
__device__ __forceinline__ unsigned dilate3(unsigned v) {
    v = (v | (v << 16)) & 0x030000ffu;
    v = (v | (v << 8)) & 0x0300f00fu;
    v = (v | (v << 4)) & 0x030c30c3u;
    return (v | (v << 2)) & 0x09249249u;
}

// Sum of two deposited values modulo 2^popcount(mask): with the bits outside the
// mask set to one, carries run through them to the next mask bit.
__device__ __forceinline__ unsigned long long dilated_add(unsigned long long x, unsigned long long y,
                                                          unsigned long long mask) {
    return ((x | ~mask) + y) & mask;
}

// Difference of two deposited values modulo 2^popcount(mask): borrows run
// through the zero bits outside the mask.
__device__ __forceinline__ unsigned long long dilated_sub(unsigned long long x, unsigned long long y,
                                                          unsigned long long mask) {
    return (x - y) & mask;
}

// per-wave LDS of the cell enumeration: per axis and offset t = 0..63 from the
// range's first cell, the key bits of the cell coordinate with its periodic
// image in the top bits (2 per axis: shift + 1 in box sides), and its squared
// distance from the box in units of the scan radius (rounded down)
constexpr int kImageBit = 58;
struct ScanLds {
    unsigned long long key[3][kWave];
    float dist2[3][kWave];
    int owner[kWave];       // cell of the batch whose particles start at each slot of a chunk, or -1
};

// per-wave LDS of the group scan: the staged candidates, kStage at a time
constexpr int kStage = 256;
struct GroupLds {
    double x[kStage], y[kStage], z[kStage];   // image position next to the group
    int j[kStage];
    ScanLds cells;
};

__device__ __forceinline__ double sq_disp(const double4& q, const double xi[3], int wrap, const double box[3]) {
    double d0 = q.x - xi[0], d1 = q.y - xi[1], d2 = q.z - xi[2];
    if (wrap) {
        d0 = min_image(d0, box[0], wrap & 1);
        d1 = min_image(d1, box[1], wrap & 2);
        d2 = min_image(d2, box[2], wrap & 4);
    }
    return d0 * d0 + d1 * d1 + d2 * d2;
}

// Bit 63 - k of the mask is set when staged particle g + k lies inside the
// sphere, displacements taken at the minimum image (scans that span a periodic
// axis whole).  Slots past the staged ones hold stale values; the caller drops
// their bits.
__device__ __forceinline__ unsigned long long wrap_mask(const GroupLds& S, int g, const double xi[3], double R2,
                                                        int wrap, const double box[3]) {
    unsigned long long mk = 0;
    for (int k0 = 0; k0 < kWave; k0 += 4) {
        unsigned b = 0;
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const double4 q = make_double4(S.x[g + k0 + k], S.y[g + k0 + k], S.z[g + k0 + k], 0.0);
            b = (b << 1) + (sq_disp(q, xi, wrap, box) < R2 ? 1u : 0u);
        }
        mk = (mk << 4) | b;
    }
    return mk;
}

// ---------------------------------------------------- sphere tests on matrix cores
// |q - x|^2 - R^2 = |q|^2 - 2 q.x + (|x|^2 - R^2) is a contraction over the
// components of the candidate q and the particle x: 32 candidates against 32
// particles are one 32x32x16 FP16 matrix product, whose signs are the tests.
// Coordinates are taken relative to the group's centre, scaled so that the
// group's reach is kTestReach, and split into two FP16 parts each (22 bits);
// the K = 16 products of one pair are
//   hi.hi (3) + hi.lo (3) + lo.hi (3) + lo.lo (3) + |q|^2 (hi, lo) + t (hi, lo),
// t = |x|^2 - R^2 - kTestSlack.  Rounding: 2 x 3 x kTestReach x (the residual
// 2^-22 kTestReach of each split, both sides) for the products, 2^-22 of
// |q|^2, |x|^2 <= 3 kTestReach^2 for the two squares and about as much for the
// FP32 sums, together below 0.02; the slack of 0.14 (a few 1e-4 of R^2 for
// particles whose radii are alike) keeps every true hit, and the exact FP64
// test of the hit loop drops the rest.
constexpr float kTestReach = 48.0f;
constexpr float kTestSlack = 0.14f;
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float16v __attribute__((ext_vector_type(16)));
typedef unsigned uint4v __attribute__((ext_vector_type(4)));

union Frag {
    uint4v u;
    half8 h;
};

// Fragments of 64 points, one per lane: k 0-7 in f0 and k 8-15 in f1 of the
// lane's own point become the operands of points 0-31 (f0) and 32-63 (f1):
// lanes 0-31 hold k 0-7 and lanes 32-63 hold k 8-15 of the tile's points.
__device__ __forceinline__ void tile_fragments(Frag& f0, Frag& f1) {
#pragma unroll
    for (int c = 0; c < 4; c++) {
        unsigned a = f0.u[c], b = f1.u[c];
        swap_halves(a, b);
        f0.u[c] = a;
        f1.u[c] = b;
    }
}

__device__ __forceinline__ void split16(float v, _Float16& hi, _Float16& lo) {
    hi = (_Float16)v;
    lo = (_Float16)(v - (float)hi);
}

// candidates: (hi xyz, hi xyz, lo xy | lo z, lo xyz, |q|^2 hi, lo, 1, 1)
__device__ __forceinline__ void candidate_fragments(float x, float y, float z, Frag& f0, Frag& f1) {
    _Float16 xh, xl, yh, yl, zh, zl, qh, ql;
    split16(x, xh, xl);
    split16(y, yh, yl);
    split16(z, zh, zl);
    split16(x * x + y * y + z * z, qh, ql);
    f0.h = half8{xh, yh, zh, xh, yh, zh, xl, yl};
    f1.h = half8{zl, xl, yl, zl, qh, ql, (_Float16)1.0f, (_Float16)1.0f};
    tile_fragments(f0, f1);
}

// particles: -2 x in the slots that meet those, and t
__device__ __forceinline__ void particle_fragments(float x, float y, float z, float r2, Frag& f0, Frag& f1) {
    _Float16 xh, xl, yh, yl, zh, zl, th, tl;
    split16(-2.0f * x, xh, xl);
    split16(-2.0f * y, yh, yl);
    split16(-2.0f * z, zh, zl);
    split16(x * x + y * y + z * z - r2 - kTestSlack, th, tl);
    f0.h = half8{xh, yh, zh, xl, yl, zl, xh, yh};
    f1.h = half8{zh, xl, yl, zl, (_Float16)1.0f, (_Float16)1.0f, th, tl};
    tile_fragments(f0, f1);
}

// The signs of one product: lane l holds column l % 32 (a particle), rows
// 8 (i / 4) + 4 (l / 32) + i % 4, i = 0..15; bit 15 - i of the result is set
// where row i's value is negative.
__device__ __forceinline__ unsigned sign_bits(const Frag& cand, const Frag& part) {
    float16v d = {};
    d = __builtin_amdgcn_mfma_f32_32x32x16_f16(cand.h, part.h, d, 0, 0, 0);
    unsigned m = 0;
#pragma unroll
    for (int i = 0; i < 16; i++) m = __builtin_amdgcn_alignbit(m, (unsigned)__float_as_int(d[i]), 31);
    return m;
}

// the candidate of its tile that sits in row r of the product, so that the rows
// a half of the wave receives are 16 candidates in staging order
__device__ __forceinline__ int row_candidate(int r) { return 16 * ((r >> 2) & 1) + 4 * (r >> 3) + (r & 3); }

// Cell enumeration and staging shared by the cooperative scans: the cells of
// one table level within Rq of the box [bmin, bmax] (the finest level whose
// cells are at least scale Rq wide, kScanScale by default) are taken 64 at a
// time, one per lane (key, table entry, periodic image), and their particles
// are handed out 64 at a time, one per lane, with coalesced loads: chunk(q,
// valid, nb, wrap) runs on
// every lane for each such chunk, q being the lane's particle moved to the
// periodic image next to the box (index bits in q.w), valid whether the lane
// holds one, nb how many lanes do.  `wrap` has bit d set when the scan spans
// periodic axis d whole; displacements along such an axis must then take the
// minimum image themselves.  bmin, bmax and Rq must be uniform over the wave,
// with Rq below half of every periodic side.
// With WHOLE false a scan that would span an axis whole is not made: the result
// says whether it was.
template <bool WHOLE = true, typename Chunk>
__device__ __forceinline__ bool scan_cells(const TreeDesc& td, const int2* __restrict__ tab,
                                           const double4* __restrict__ pos, ScanLds& S, int lane,
                                           const double bmin[3], const double bmax[3], double Rq, Chunk&& chunk,
                                           double scale = kScanScale) {
    int L = td.bmax;
    while (L > 0 && fmin(td.cs[L][0], fmin(td.cs[L][1], td.cs[L][2])) < scale * Rq) L--;
    L = __builtin_amdgcn_readfirstlane(L);
    int a[3], cnt[3], wrap;
    // (a range wider than the tables takes the next coarser level)
    for (;; L--) {
        wrap = 0;
        bool wide = false;
#pragma unroll
        for (int d = 0; d < 3; d++) {
            const double s = td.cs[L][d];
            const int nc = td.ncell[L][d];
            int lo = (int)floor((bmin[d] - Rq) / s);
            int hi = (int)floor((bmax[d] + Rq) / s);
            if (td.periodic[d]) {
                if (hi - lo + 1 >= nc) {
                    lo = 0;
                    hi = nc - 1;
                    wrap |= 1 << d;
                }
            } else {
                lo = max(lo, 0);
                hi = min(hi, nc - 1);
            }
            a[d] = __builtin_amdgcn_readfirstlane(lo);
            cnt[d] = __builtin_amdgcn_readfirstlane(hi - lo + 1);
            wide |= cnt[d] > kWave;
        }
        if (!wide || L == 0) break;
    }
    wrap = __builtin_amdgcn_readfirstlane(wrap);
    if (!WHOLE && wrap) return false;
    if (cnt[0] <= 0 || cnt[1] <= 0 || cnt[2] <= 0) return true;
    const int ncells = cnt[0] * cnt[1] * cnt[2];
    // slack for the rounding of cell edges, of the keys' quantisation and of the distances in FP32
    const double Rg = Rq * (1.0 + 1e-9) + 1e-12 * fmax(td.box[0], fmax(td.box[1], td.box[2])), iRg = 1.0 / Rg;
    const float Rg2 = 1.000001f;
    // Sides of one length up to ten levels deep have every third bit each: the bits
    // are spread in 12 instructions an axis (deposit_bits takes 11 for each bit)
    const bool even = L <= 10 && td.qbits[0] == td.qbits[1] && td.qbits[0] == td.qbits[2];
    wave_lds_sync();
#pragma unroll
    for (int d = 0; d < 3; d++) {
        const int nc = td.ncell[L][d], u = a[d] + lane;
        // unwrapped cell coordinates stay within one box side of [0, nc)
        const unsigned long long image = u < 0 ? 0 : u >= nc ? 2 : 1;
        const double s = td.cs[L][d], clo = u * s;
        const double g = (wrap >> d) & 1 ? 0.0 : fmax(0.0, fmax(clo - bmax[d], bmin[d] - (clo + s)));
        const unsigned v = (unsigned)u & (nc - 1);
        const unsigned long long bits = even ? dilate3(v) << (2 - d) : deposit_bits(v, td.mask[L][d]);
        S.key[d][lane] = bits | (image << (kImageBit + 2 * d));
        const float q = (float)(g * iRg);
        S.dist2[d][lane] = q * q * 0.9999998f;
    }
    wave_lds_sync();
    const int2* __restrict__ cells = tab + td.tab_off[L];
    // cell coordinates from the flat index through FP32 reciprocals (exact for
    // the few thousand cells a scan covers)
    const float inv2 = 1.0f / (float)cnt[2], inv1 = 1.0f / (float)cnt[1];
    for (int c0 = 0; c0 < ncells; c0 += kWave) {
        const int c = c0 + lane;
        int num = 0, st = 0, img = 0;
        if (c < ncells) {
            const int t = (int)(((float)c + 0.5f) * inv2);
            const int tz = c - t * cnt[2];
            const int tx = (int)(((float)t + 0.5f) * inv1);
            const int ty = t - tx * cnt[1];
            if (S.dist2[0][tx] + S.dist2[1][ty] + S.dist2[2][tz] < Rg2) {
                const unsigned long long key = S.key[0][tx] | S.key[1][ty] | S.key[2][tz];
                const int2 se = cells[key & ((1ull << kImageBit) - 1)];
                st = se.x;
                num = se.y - se.x;
                img = (int)(key >> kImageBit);
            }
        }
        const int incl = wave_prefix_sum(num), excl = incl - num;
        const int total = __builtin_amdgcn_readlane(incl, kWave - 1);
        for (int t0 = 0; t0 < total; t0 += kWave) {
            // each cell with particles in the chunk marks its first slot there;
            // the last mark at or below a slot is the cell that holds it
            S.owner[lane] = -1;
            wave_lds_sync();
            if (num > 0 && incl > t0 && excl < t0 + kWave) S.owner[max(excl - t0, 0)] = lane;
            wave_lds_sync();
            const int k = wave_prefix_max(S.owner[lane]);
            const int t = t0 + lane;
            const int j = __shfl(st - excl, k, kWave) + t, im = __shfl(img, k, kWave);
            // lanes past the end hold a far-away point that no sphere reaches
            double4 q = make_double4(1e30, 1e30, 1e30, __longlong_as_double(-1ll));
            if (t < total) {
                const double4 p = pos[j];
                // shifts of -1, 0 or 1 box sides (the product is exact)
                q = make_double4(p.x + (double)((im & 3) - 1) * td.box[0], p.y + (double)(((im >> 2) & 3) - 1) * td.box[1],
                                 p.z + (double)((im >> 4) - 1) * td.box[2], __longlong_as_double((long long)j));
            }
            chunk(q, t < total, min(kWave, total - t0), wrap);
            wave_lds_sync();   // the next chunk overwrites the owners
        }
    }
    return true;
}

// The lanes one group scan serves: of the lanes that still need one, those with
// a radius of at least kClassRatio times the largest, within kClassWindow times
// that of the first of them on every axis; their box and largest radius.
// Fewer, wider classes pay down to a quarter: each pass scans the union once,
// and its narrow lanes' extra candidates cost less than passes of their own.
constexpr double kClassRatio = 0.25;
constexpr double kClassWindow = 2.0;
struct ScanClass {
    bool in;
    double Rq, bmin[3], bmax[3];
};
__device__ __forceinline__ ScanClass scan_class(bool need, double R, const double xi[3]) {
    ScanClass c;
    const double Rref = uniform_d(wave_max_d(need ? R : 0.0));
    const bool big = need && R >= kClassRatio * Rref;
    const int leader = __builtin_amdgcn_readfirstlane(__ffsll((long long)__ballot(big)) - 1);
    const double win = kClassWindow * Rref;
    bool in = big;
#pragma unroll
    for (int d = 0; d < 3; d++) {
        const double xl = uniform_d(__shfl(xi[d], leader, kWave));
        in &= fabs(xi[d] - xl) <= win;
    }
    c.in = in;
    c.Rq = uniform_d(wave_max_d(in ? R : 0.0));
#pragma unroll
    for (int d = 0; d < 3; d++) {
        c.bmin[d] = uniform_d(wave_min_d(in ? xi[d] : INFINITY));
        c.bmax[d] = uniform_d(wave_max_d(in ? xi[d] : -INFINITY));
    }
    return c;
}

// Tests every particle of every cell within Rq + pad of the box [bmin, bmax]
// against the calling lane's sphere |x - xi|^2 < R2 (R2 <= Rq^2; lanes with sel
// false take no hits) and calls hit(j, r2) for each particle inside, in the
// order the cells are scanned.  The candidates are staged in LDS, kStage at a
// time across cell batches; a full stage is tested on the matrix cores, 64
// candidates against the wave's 64 particles with four products (about 1.7
// vector instructions per 64 tests, where testing each in FP64 took 10), into
// 64-bit masks per lane.  The lanes then walk the set bits of the whole stage
// together: the lanes' hits are spread unevenly over the candidates, and a lane
// waits for the busiest one once per stage, not once per 64 candidates.
// Measured with both (solve stage): clustered 16.8M particles 44.6 -> 36.8 ms,
// jittered lattice 2.1M 1.79 -> 1.41 ms.
// (WHOLE as in scan_cells)
template <bool WHOLE, typename Hit>
__device__ __forceinline__ bool group_scan(const TreeDesc& td, const int2* __restrict__ tab,
                                           const double4* __restrict__ pos, GroupLds& S, int lane,
                                           const double bmin[3], const double bmax[3], double Rq, double pad,
                                           const double xi[3], double R2, bool sel, Hit&& hit) {
    // the test frame: relative to the box's centre, the reach of the group's
    // spheres scaled to kTestReach; candidates beyond the reach on an axis are
    // moved to just beyond it, where no sphere comes
    const double cen[3] = {0.5 * (bmin[0] + bmax[0]), 0.5 * (bmin[1] + bmax[1]), 0.5 * (bmin[2] + bmax[2])};
    const double reach = 0.5 * fmax(bmax[0] - bmin[0], fmax(bmax[1] - bmin[1], bmax[2] - bmin[2])) + 1.01 * Rq;
    const double scale = (double)kTestReach / reach;
    Frag p0, p1;
    particle_fragments((float)((xi[0] - cen[0]) * scale), (float)((xi[1] - cen[1]) * scale),
                       (float)((xi[2] - cen[2]) * scale), (float)(R2 * (scale * scale)), p0, p1);
    const int row = (lane & 32) + row_candidate(lane & 31);
    int ns = 0;      // staged candidates
    int spans = 0;   // axes the scan spans whole
    auto drain = [&]() {
        wave_lds_sync();
        constexpr int kWords = kStage / 32;
        unsigned mk[kWords] = {};   // bit 31 - b of word w: staged candidate 32 w + b
        int left = 0;
#pragma unroll 1
        for (int g = 0; g < kStage; g += kWave) {
            unsigned long long m = 0;
            if (g < ns) {
                if (WHOLE && spans) {
                    m = wrap_mask(S, g, xi, R2, spans, td.box);
                } else {
                    float f[3] = {(float)((S.x[g + row] - cen[0]) * scale), (float)((S.y[g + row] - cen[1]) * scale),
                                  (float)((S.z[g + row] - cen[2]) * scale)};
#pragma unroll
                    for (int d = 0; d < 3; d++) f[d] = fminf(kTestReach, fmaxf(-kTestReach, f[d]));
                    Frag c0, c1;
                    candidate_fragments(f[0], f[1], f[2], c0, c1);
                    unsigned a0 = sign_bits(c0, p0), a1 = sign_bits(c0, p1);
                    swap_halves(a0, a1);   // the lane's own particle: candidates 0-15, 16-31
                    unsigned b0 = sign_bits(c1, p0), b1 = sign_bits(c1, p1);
                    swap_halves(b0, b1);   // 32-47, 48-63
                    m = ((unsigned long long)((a0 << 16) | a1) << 32) | ((b0 << 16) | b1);
                }
                if (ns - g < kWave) m &= ~(~0ull >> (ns - g));
                if (!sel) m = 0;
            }
            left += __popcll(m);
#pragma unroll
            for (int q = 0; q + 2 < kWords; q++) mk[q] = mk[q + 2];
            mk[kWords - 2] = (unsigned)(m >> 32);
            mk[kWords - 1] = (unsigned)m;
        }
        int base = -32;
        unsigned cur = 0;
        while (left > 0) {
            while (cur == 0) {
                cur = mk[0];
                base += 32;
#pragma unroll
                for (int q = 0; q + 1 < kWords; q++) mk[q] = mk[q + 1];
            }
            const int b = __builtin_clz(cur);
            cur &= 0x7fffffffu >> b;
            left--;
            const int k = base + b;
            const double r2 = sq_disp(make_double4(S.x[k], S.y[k], S.z[k], 0.0), xi, WHOLE ? spans : 0, td.box);
            if (r2 < R2) hit(S.j[k], r2);
        }
        wave_lds_sync();   // the next candidates overwrite the stage
        ns = 0;
    };
    const bool made = scan_cells<WHOLE>(td, tab, pos, S.cells, lane, bmin, bmax, Rq + pad, [&](const double4& q, bool valid, int nb, int wrap) {
        spans = wrap;
        if (ns + nb > kStage) drain();
        if (valid) {
            S.x[ns + lane] = q.x;
            S.y[ns + lane] = q.y;
            S.z[ns + lane] = q.z;
            S.j[ns + lane] = (int)__double_as_longlong(q.w);
        }
        ns += nb;
    });
    if (ns > 0) drain();
    return made;
}

}  // namespace mfm
