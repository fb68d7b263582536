// Learned warm start (beyond the paper): per-atom features from the 16
// nearest atoms of the same system, a 3-layer perceptron (BF16 weights and
// activations, FP32 accumulation on the matrix cores) that predicts a
// displacement of every atom, its training kernels, and the application of
// the displacement before a minimization.  The minimizer keeps the last word: a
// displaced start is kept per system only where the energy prefers it.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <string>

#include "ff.h"
#include "ff_learn.h"

namespace ff {

// ------------------------------------------------------------------ BF16
// Round to nearest even from FP32 (values here are finite).
__device__ __forceinline__ uint16_t to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// ------------------------------------------------------------- features
// Row i of the features:
//   f[0..2]          = q, sigma - 3.5, 10 eps of the atom,
//   f[3+7k .. 9+7k]  = (x_j - x_i)/4 (3 values), r/4, q_j, sigma_j - 3.5, 10 eps_j
// for its k-th nearest other atom of the same system by FP64 squared distance
// (ties to the lower index; zeros for missing neighbours), then the place of
// the atom in its system: (x_i - c)/16 (3 values) and |x_i - c|/16 with c the
// centroid (a sum in atom order divided by n), and n/4096; zeros up to
// FF_LEARN_FEATURES.  Each value is rounded FP64 -> FP32 -> BF16.
//
// One launch of two kinds of workgroups that write disjoint bytes:
//  - one per system or group of small systems sums coordinates in atom order and
//    writes the three offsets and their length of every row (centroid_rows,
//    centroid_group);
//  - one per 16 atoms, each of its wavefronts searching the neighbours of four
//    (neighbor_rows).
constexpr int kPlace = 3 + 7 * FF_LEARN_NEIGHBORS;   // first entry of an atom's place in its system
constexpr int kKnnTile = 256;                        // atoms staged in LDS at a time
constexpr int kKnnLoads = 3 * kKnnTile / 256;        // ... by so many 8-byte loads of each thread

// DPP move within each row of 16 lanes.
template <int CTRL, int BANKS = 0xF>
__device__ __forceinline__ int row_move(int old, int v) {
    return __builtin_amdgcn_update_dpp(old, v, CTRL, 0xF, BANKS, false);
}
// Value of lane (rank ^ X) of the row.
template <int X>
__device__ __forceinline__ int row_xor(int v) {
    static_assert(X == 1 || X == 2 || X == 3 || X == 4 || X == 7 || X == 8 || X == 15, "rows of 16 lanes");
    if (X == 1) return row_move<0xB1>(v, v);            // quad_perm [1,0,3,2]
    if (X == 2) return row_move<0x4E>(v, v);            // quad_perm [2,3,0,1]
    if (X == 3) return row_move<0x1B>(v, v);            // quad_perm [3,2,1,0]
    if (X == 4) return row_move<0x114, 0xA>(row_move<0x104, 0x5>(v, v), v);   // row_shl:4 / row_shr:4 by banks
    if (X == 7) return row_move<0x141>(v, v);           // row_half_mirror
    if (X == 8) return row_move<0x128>(v, v);           // row_ror:8
    return row_move<0x140>(v, v);                       // row_mirror
}
template <int X>
__device__ __forceinline__ double row_xor(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = row_xor<X>((int)(b & 0xffffffffLL)), hi = row_xor<X>((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// One (distance, index) entry per lane, ordered by distance, then index.
struct Near { double d; int j; };
__device__ __forceinline__ bool nearer(const Near& a, const Near& b) {
    return (a.d < b.d) | ((a.d == b.d) & (a.j < b.j));
}
// Compare-exchange of ranks r and r ^ X: the lower rank keeps the nearer entry.
template <int X>
__device__ __forceinline__ void order_ranks(Near& e, int rank) {
    const Near o{row_xor<X>(e.d), row_xor<X>(e.j)};
    constexpr int top = X >= 8 ? 8 : (X >= 4 ? 4 : (X >= 2 ? 2 : 1));     // highest bit of X
    const bool take = nearer(o, e) != ((rank & top) != 0);
    e.d = take ? o.d : e.d;
    e.j = take ? o.j : e.j;
}
// Sorts the 16 entries of each row (bitonic, ten exchanges) and merges them
// into the row's sorted list, of which the 16 nearest stay (five more).
__device__ __forceinline__ void merge_row(Near& list, Near e, int rank) {
    order_ranks<1>(e, rank);
    order_ranks<3>(e, rank);
    order_ranks<1>(e, rank);
    order_ranks<7>(e, rank);
    order_ranks<2>(e, rank);
    order_ranks<1>(e, rank);
    order_ranks<15>(e, rank);
    order_ranks<4>(e, rank);
    order_ranks<2>(e, rank);
    order_ranks<1>(e, rank);
    const Near o{row_xor<15>(e.d), row_xor<15>(e.j)};
    const bool take = nearer(o, list);
    list.d = take ? o.d : list.d;
    list.j = take ? o.j : list.j;
    order_ranks<8>(list, rank);
    order_ranks<4>(list, rank);
    order_ranks<2>(list, rank);
    order_ranks<1>(list, rank);
}

__device__ __forceinline__ double lane_value(double v, int lane) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffLL), lane);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Sums of the workgroup's 256 threads, in every thread.
__device__ __forceinline__ double block_total(double v, double* red) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return (red[0] + red[1]) + (red[2] + red[3]);
}

// The coordinates of system [j0, j1) summed one by one in atom order: three
// lanes carry the running sums (x, y, z) over tiles that the whole workgroup
// stages in LDS, the next tile's loads in flight meanwhile.  Bound by a chain
// of n dependent FP64 additions (8 ns each).
__device__ void ordered_sum(const double* __restrict__ x, int n, double (*tile)[3 * kKnnTile], double (&sum)[3]) {
    const int t = threadIdx.x, n_el = 3 * n;
    double s = 0.0;
    double v[kKnnLoads];
#pragma unroll
    for (int c = 0; c < kKnnLoads; ++c) v[c] = t + c * 256 < n_el ? x[t + c * 256] : 0.0;
    int buf = 0;
    for (int a0 = 0; a0 < n; a0 += kKnnTile, buf ^= 1) {
#pragma unroll
        for (int c = 0; c < kKnnLoads; ++c) tile[buf][t + c * 256] = v[c];
        __syncthreads();
        const int e0 = 3 * (a0 + kKnnTile) + t;
#pragma unroll
        for (int c = 0; c < kKnnLoads; ++c) v[c] = e0 + c * 256 < n_el ? x[e0 + c * 256] : 0.0;
        if (t < 3) {
            const double* p = tile[buf] + t;
            const int m = min(kKnnTile, n - a0);
            int a = 0;
            for (; a + 16 <= m; a += 16) {
                double w[16];
#pragma unroll
                for (int k = 0; k < 16; ++k) w[k] = p[3 * (a + k)];
#pragma unroll
                for (int k = 0; k < 16; ++k) s += w[k];
            }
            for (; a < m; ++a) s += p[3 * a];
        }
    }
    __syncthreads();
    if (t < 3) tile[0][t] = s;
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 3; ++c) sum[c] = tile[0][c];
}

// Place entries of the rows first, first + stride, ... of a system of n atoms, from
// its coordinate sums.  With err > 0 the sums may be off by that much from the ordered ones: the
// return value says whether an entry of this thread's rows could then round
// to another BF16 value.
__device__ __forceinline__ bool place_rows(const double* __restrict__ x, int n, const double (&sum)[3], double err,
                           uint16_t* __restrict__ feat, int first = threadIdx.x, int stride = 256) {
#pragma clang fp contract(off)
    const double nd = (double)n;
    const double c0 = sum[0] / nd, c1 = sum[1] / nd, c2 = sum[2] / nd;
    bool unsure = false;
#pragma unroll 4
    for (int a = first; a < n; a += stride) {
        const double px = x[3 * (size_t)a], py = x[3 * (size_t)a + 1], pz = x[3 * (size_t)a + 2];
        const double cx = px - c0, cy = py - c1, cz = pz - c2;
        const double v[4] = {cx / 16.0, cy / 16.0, cz / 16.0, sqrt(cx * cx + cy * cy + cz * cz) / 16.0};
        uint16_t* h = feat + (size_t)a * FF_LEARN_FEATURES + kPlace;
        // sum error through the division, the difference, the length and /16
        // (and the rounding of each)
        const double e = 0.25 * (err / nd) +
                         0x1p-48 * (fabs(px) + fabs(py) + fabs(pz) + fabs(c0) + fabs(c1) + fabs(c2));
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint16_t b = to_bf16((float)v[k]);
            h[k] = b;
            if (err > 0.0) unsure |= to_bf16((float)(v[k] - e)) != b || to_bf16((float)(v[k] + e)) != b;
        }
    }
    return unsure;
}

// The centroid is defined by the ordered sum, whose dependent additions would
// take longer than the neighbour search beside it (80 us at 10,000 atoms), but
// only BF16 roundings of its offsets are wanted.  So the workgroup sums in
// parallel and bounds the difference: either order is within n u sum|x| of
// the exact sum (u = 2^-53), so they differ by less than err = n 2^-51 sum|x|.
// Where every entry rounds alike over that range the rows hold what the
// ordered sum gives; else (some 1e-3 of 10,000-atom systems) it is formed.
__device__ __forceinline__ void centroid_rows(const double* __restrict__ xyz, int j0, int j1, uint16_t* __restrict__ feat,
                              double (*tile)[3 * kKnnTile]) {
#pragma clang fp contract(off)
    const int t = threadIdx.x, n = j1 - j0, n_el = 3 * n;
    if (n < 1) return;
    const double* x = xyz + 3 * (size_t)j0;
    uint16_t* rows = feat + (size_t)j0 * FF_LEARN_FEATURES;
    // elements t + 256 (3 k + c) of the flat array are component (t + c) mod 3
    double part[3] = {0.0, 0.0, 0.0}, mag = 0.0;
#pragma unroll 4
    for (int e = t; e < n_el; e += 3 * 256)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double v = e + c * 256 < n_el ? x[e + c * 256] : 0.0;
            part[c] += v;
            mag += fabs(v);
        }
    const int r = t % 3;
    double sum[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) sum[c] = block_total(r == c ? part[0] : ((r + 1) % 3 == c ? part[1] : part[2]), tile[0]);
    const double err = block_total(mag, tile[0]) * ((double)n * 0x1p-51);
    __syncthreads();
    bool unsure = !(err > 0.0 && err <= __DBL_MAX__);
    if (!unsure) unsure = place_rows(x, n, sum, err, rows);
    if (!__syncthreads_or(unsure)) return;
    ordered_sum(x, n, tile, sum);
    place_rows(x, n, sum, 0.0, rows);
}

// The same for a system of at most W atoms by W lanes of a wavefront (n and j0
// may differ between the wavefront's groups of W): a lane holds an atom, and the
// sum is formed in order.
template <int W>
__device__ __forceinline__ void centroid_lanes(const double* __restrict__ xyz, int j0, int n, uint16_t* __restrict__ feat) {
    const int l = threadIdx.x & (W - 1);
    double p[3] = {0.0, 0.0, 0.0}, sum[3] = {0.0, 0.0, 0.0};
    if (l < n)
#pragma unroll
        for (int c = 0; c < 3; ++c) p[c] = xyz[3 * (size_t)(j0 + l) + c];
    for (int a = 0; __any(a < n); ++a)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double v = W == 64 ? lane_value(p[c], a) : __shfl(p[c], a, W);
            if (a < n) sum[c] += v;
        }
    if (n > 0) place_rows(xyz + 3 * (size_t)j0, n, sum, 0.0, feat + (size_t)j0 * FF_LEARN_FEATURES, l, W);
}

// Systems [s0, s0 + kGroup) by one workgroup: 16 lanes, a wavefront or the whole
// workgroup for each, as their sizes ask.
constexpr int kGroup = 16;
__device__ __forceinline__ void centroid_group(const double* __restrict__ xyz, const int32_t* __restrict__ sys_first,
                                               int s0, int n_sys, uint16_t* __restrict__ feat,
                                               double (*tile)[3 * kKnnTile]) {
    auto first = [&](int s) { return s < n_sys ? sys_first[s] : 0; };
    auto size = [&](int s) { return s < n_sys ? sys_first[s + 1] - sys_first[s] : 0; };
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), own = s0 + (threadIdx.x >> 4);
    centroid_lanes<16>(xyz, first(own), size(own) <= 16 ? size(own) : 0, feat);
    for (int s = s0 + 4 * wave; s < s0 + 4 * wave + 4; ++s)
        if (size(s) > 16 && size(s) <= 64) centroid_lanes<64>(xyz, first(s), size(s), feat);
    for (int s = s0; s < s0 + kGroup; ++s)
        if (size(s) > 64) centroid_rows(xyz, first(s), first(s) + size(s), feat, tile);
}

// Neighbours and row entries of atoms [a0, a0 + 16), four per wavefront.  A
// lane takes one candidate of 64 at a time for each of the four atoms; those
// not farther than an atom's 16th nearest so far go to its queue in LDS.  Once
// a queue holds 16, the last 16 of every queue are merged into the atoms'
// lists, which lie sorted in the 16 lanes of row k for atom k: one merge
// serves four atoms.  The order is total (distance, then index), so the
// result does not depend on the order of candidates, and the search starts
// around the atoms themselves: chain neighbours set a tight limit before the rest is
// scanned.
// Bound by VALU issue of the first pass (30 instructions per 64 candidates and
// four atoms) and below a few thousand atoms by latency.  10,000 atoms: 67 us,
// against 1.81 ms for one thread per atom scanning every candidate, which left
// 157 wavefronts on 1,024 SIMDs; 50,000 atoms 0.73 ms, 300 atoms 14 us.
// Inserting candidates one by one through scalar registers instead of merging
// 16 took 2-3 times as long below 4,000 atoms; testing all of them in FP64,
// without the FP32 pass, 0.99 ms at 50,000 atoms.
constexpr int kKnnAtoms = 4;                         // atoms per wavefront: one per row of 16 lanes
constexpr int kKnnQueue = 64 + 16;                   // candidates waiting per atom: at most 15 + 64

template <bool MANY>
__device__ __forceinline__ void neighbor_rows(const double* __restrict__ xyz, const double* __restrict__ q,
                              const double* __restrict__ sig, const double* __restrict__ eps,
                              const int32_t* __restrict__ sys_first, const int32_t* __restrict__ atom_sys, int a0,
                              int n_total, uint16_t* __restrict__ feat, int32_t* __restrict__ nbr,
                              double (*tile)[3 * kKnnTile], double* __restrict__ queue_d,
                              int* __restrict__ queue_j, uint16_t* __restrict__ rowbuf) {
#pragma clang fp contract(off)
    constexpr int A = kKnnAtoms;
    const int t = threadIdx.x, lane = t & 63, rank = t & 15, row = (t & 63) >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int last = min(a0 + 4 * A, n_total) - 1;
    const int s_lo = atom_sys[a0], s_hi = atom_sys[last];
    const int lo = sys_first[s_lo], hi = sys_first[s_hi + 1];   // candidates of all of the workgroup's atoms
    const bool mixed = s_lo != s_hi;                            // ... which then differ from atom to atom
    const int n_c = hi - lo, n_el = 3 * n_c;
    const int n_tiles = (n_c + kKnnTile - 1) / kKnnTile;
    const double* x = xyz + 3 * (size_t)lo;
    int ai[A], jb[A], je[A];
    double xi[A], yi[A], zi[A], limit[A];
#pragma unroll
    for (int k = 0; k < A; ++k) {
        const int i = min(a0 + wave * A + k, n_total - 1);      // (rows past the end are not written)
        const int s = mixed ? atom_sys[i] : s_lo;
        ai[k] = i - lo;
        jb[k] = sys_first[s] - lo;
        je[k] = sys_first[s + 1] - lo;
        xi[k] = xyz[3 * (size_t)i]; yi[k] = xyz[3 * (size_t)i + 1]; zi[k] = xyz[3 * (size_t)i + 2];
        limit[k] = __DBL_MAX__;                                 // candidates have finite distances
    }
    Near list{__builtin_inf(), -1};                             // entry `rank` of row's atom
    double* qd = queue_d + wave * A * kKnnQueue;
    int* qj = queue_j + wave * A * kKnnQueue;
    int waiting[A] = {};
    // the last 16 entries of every queue (missing ones: infinity) into the lists
    auto merge = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        int at = 0, end = 0;
#pragma unroll
        for (int k = 0; k < A; ++k) {
            const int first = max(waiting[k] - 16, 0);
            at = row == k ? first : at;
            end = row == k ? waiting[k] : end;
            waiting[k] = first;
        }
        at += rank;
        Near e{__builtin_inf(), -1};
        if (at < end) e = Near{qd[row * kKnnQueue + at], qj[row * kKnnQueue + at]};
        merge_row(list, e, rank);
#pragma unroll
        for (int k = 0; k < A; ++k) limit[k] = fmin(lane_value(list.d, 16 * k + 15), __DBL_MAX__);
    };
    // First pass: FP32 tests |x_j|^2 - 2 x_i.x_j <= limit - |x_i|^2 in
    // coordinates relative to the wavefront's first atom.  A candidate at
    // distance d <= r = sqrt(limit) of atom i, itself ro from the first, lies
    // within r + ro of it, so coordinates, products and sums round by less than
    // 2^-18 (r + 2 ro)^2 in all: the test with that margin misses none.
    float xf[A], yf[A], zf[A], bound[A];
    double ro[A];
#pragma unroll
    for (int k = 0; k < A; ++k) {
        const double dx = xi[k] - xi[0], dy = yi[k] - yi[0], dz = zi[k] - zi[0];
        xf[k] = (float)(-2.0 * dx); yf[k] = (float)(-2.0 * dy); zf[k] = (float)(-2.0 * dz);
        ro[k] = dx * dx + dy * dy + dz * dz;
        bound[k] = __builtin_inff();
    }
    auto pass_bounds = [&]() {
#pragma unroll
        for (int k = 0; k < A; ++k) {
            const double r = sqrt(limit[k]) + 2.0 * sqrt(ro[k]);
            // (+: FP32 underflow; beyond 2^60 squares may exceed FP32, and every candidate passes)
            bound[k] = r < 0x1p60 ? (float)(limit[k] - ro[k] + 0x1p-18 * (r * r)) + 0x1p-100f : __builtin_inff();
        }
    };
    // candidate c is atom (start + c) mod n_c: the first tile lies around the
    // workgroup's atoms.  The loads of the next two tiles are in flight (without
    // a branch around them: the wait for one must not include the next);
    // candidates past the end are NaN, which the second pass never admits.
    const int start = max(0, min(a0 - lo - (kKnnTile - 16) / 2, n_c - kKnnTile));
    auto load = [&](int step, double (&v)[kKnnLoads]) {
        const int e0 = 3 * kKnnTile * step + t;
#pragma unroll
        for (int c = 0; c < kKnnLoads; ++c) {
            const int e = min(e0 + c * 256, n_el - 1) + 3 * start;
            v[c] = x[e >= n_el ? e - n_el : e];
        }
    };
    auto scan = [&](int step, double (&v)[kKnnLoads]) {
        const int base = step * kKnnTile, buf = step & 1;
#pragma unroll
        for (int c = 0; c < kKnnLoads; ++c)
            tile[buf][c * 256 + t] = 3 * base + c * 256 + t < n_el ? v[c] : __builtin_nan("");
        __syncthreads();
        load(step + 2, v);
        // first pass: which 64 candidates may hold one for any of the four atoms
        // (where a window of candidates is one 64: that one)
        unsigned hit = MANY && n_c <= 64 ? 1u : 0u;
        if (!MANY || hit == 0)
#pragma unroll
        for (int no = 0; no < kKnnTile / 64; ++no) {
            const double* p = tile[buf] + 3 * (no * 64 + lane);
            const float xj = (float)(p[0] - xi[0]), yj = (float)(p[1] - yi[0]), zj = (float)(p[2] - zi[0]);
            const float rr = __fmaf_rn(zj, zj, __fmaf_rn(yj, yj, xj * xj));
            bool near = false;
#pragma unroll
            for (int k = 0; k < A; ++k)
                near |= !(__fmaf_rn(zf[k], zj, __fmaf_rn(yf[k], yj, __fmaf_rn(xf[k], xj, rr))) > bound[k]);
            hit |= (__ballot(near) && base + no * 64 < n_c ? 1u : 0u) << no;
        }
        // second pass over those (the atoms' own first): into the queues
        const int own = step == 0 ? (ai[0] - start) >> 6 : 0;
#pragma unroll 1
        for (int s4 = 0; s4 < kKnnTile / 64; ++s4) {
            const int no = (s4 + own) & (kKnnTile / 64 - 1);
            if (!((hit >> no) & 1u)) continue;
            const int sub = no * 64, c0 = base + sub;
            const int jw = start + c0 + lane, j = jw >= n_c ? jw - n_c : jw;     // (used below n_c only)
            const double* p = tile[buf] + 3 * (sub + lane);
            const double xj = p[0], yj = p[1], zj = p[2];
            double d2[A];
            unsigned long long m[A];
#pragma unroll
            for (int k = 0; k < A; ++k) {
                const double dx = xj - xi[k], dy = yj - yi[k], dz = zj - zi[k];
                d2[k] = dx * dx + dy * dy + dz * dz;
                m[k] = __ballot(d2[k] <= limit[k]);
                const int self = (ai[k] >= start ? ai[k] - start : ai[k] - start + n_c) - c0;
                if (self >= 0 && self < 64) m[k] &= ~(1ull << self);
                if (mixed) m[k] &= __ballot(j >= jb[k] && j < je[k]);
            }
#pragma unroll
            for (int k = 0; k < A; ++k) {
                if ((m[k] >> lane) & 1ull) {
                    const int at = k * kKnnQueue + waiting[k] + __popcll(m[k] & ((1ull << lane) - 1ull));
                    qd[at] = d2[k];
                    qj[at] = j;
                }
                waiting[k] += __popcll(m[k]);
            }
            while (max(max(waiting[0], waiting[1]), max(waiting[2], waiting[3])) >= 16) merge();
        }
        if (hit) pass_bounds();
    };
    double va[kKnnLoads], vb[kKnnLoads];
    load(0, va);
    load(1, vb);
    for (int step = 0; step < n_tiles; step += 2) {
        scan(step, va);
        if (step + 1 < n_tiles) scan(step + 1, vb);
    }
    if (waiting[0] | waiting[1] | waiting[2] | waiting[3]) merge();
    // row k writes atom k's row into LDS; it is stored as 32-bit words (where
    // the array is aligned to them) but for the entries of the atom's place,
    // which the centroid workgroup writes
    uint16_t* rows = rowbuf + wave * A * FF_LEARN_FEATURES;
    const int i = a0 + wave * A + row;
    if (i <= last) {
        uint16_t* f = rows + row * FF_LEARN_FEATURES;
        uint16_t* g = f + 3 + 7 * rank;
        const int j = list.j < 0 ? -1 : lo + list.j;
        if (nbr) nbr[(size_t)i * FF_LEARN_NEIGHBORS + rank] = j;
        if (j < 0) {
            for (int c = 0; c < 7; ++c) g[c] = 0;
        } else {
            const double dx = xyz[3 * (size_t)j] - xyz[3 * (size_t)i], dy = xyz[3 * (size_t)j + 1] - xyz[3 * (size_t)i + 1],
                         dz = xyz[3 * (size_t)j + 2] - xyz[3 * (size_t)i + 2];
            g[0] = to_bf16((float)(dx / 4.0));
            g[1] = to_bf16((float)(dy / 4.0));
            g[2] = to_bf16((float)(dz / 4.0));
            g[3] = to_bf16((float)(sqrt(list.d) / 4.0));
            g[4] = to_bf16((float)q[j]);
            g[5] = to_bf16((float)(sig[j] - 3.5));
            g[6] = to_bf16((float)(10.0 * eps[j]));
        }
        const int s = mixed ? atom_sys[i] : s_lo;
        if (rank == 0) f[0] = to_bf16((float)q[i]);
        if (rank == 1) f[1] = to_bf16((float)(sig[i] - 3.5));
        if (rank == 2) f[2] = to_bf16((float)(10.0 * eps[i]));
        if (rank == 3) f[kPlace + 4] = to_bf16((float)((double)(sys_first[s + 1] - sys_first[s]) / 4096.0));
        if (rank >= 4 && rank < 4 + FF_LEARN_FEATURES - (kPlace + 5)) f[kPlace + 5 + rank - 4] = 0;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const bool words = (uintptr_t)feat % 4 == 0;
    for (int k = 0; k < A && a0 + wave * A + k <= last; ++k) {
        const uint16_t* r = rows + k * FF_LEARN_FEATURES;
        uint16_t* f = feat + (size_t)(a0 + wave * A + k) * FF_LEARN_FEATURES;
        constexpr int w_lo = kPlace / 2, w_hi = (kPlace + 4) / 2;   // first and last word shared with the place
        const bool both = lane < w_lo || lane > w_hi;
        if (both && words) {
            ((uint32_t*)f)[lane] = ((const uint32_t*)r)[lane];
            continue;
        }
        if (both || lane == w_lo) f[2 * lane] = r[2 * lane];
        if (both || lane == w_hi) f[2 * lane + 1] = r[2 * lane + 1];
    }
}

// Grid: the centroid workgroups, one per system (MANY: per kGroup systems), then
// one per 4 * kKnnAtoms atoms.
template <bool MANY>
__global__ void __launch_bounds__(256) k_features(const double* __restrict__ xyz, const double* __restrict__ q,
                                                  const double* __restrict__ sig, const double* __restrict__ eps,
                                                  const int32_t* __restrict__ sys_first,
                                                  const int32_t* __restrict__ atom_sys, int n_sys, int n_total,
                                                  uint16_t* __restrict__ feat, int32_t* __restrict__ nbr) {
    static_assert(kPlace % 2 == 1 && FF_LEARN_FEATURES == 128, "row words of the place entries");
    __shared__ double tile[2][3 * kKnnTile];
    __shared__ double queue_d[4 * kKnnAtoms * kKnnQueue];
    __shared__ int queue_j[4 * kKnnAtoms * kKnnQueue];
    __shared__ __attribute__((aligned(4))) uint16_t rowbuf[4 * kKnnAtoms * FF_LEARN_FEATURES];
    const int b = blockIdx.x, centroids = MANY ? (n_sys + kGroup - 1) / kGroup : n_sys;
    if (b >= centroids)
        neighbor_rows<MANY>(xyz, q, sig, eps, sys_first, atom_sys, (b - centroids) * 4 * kKnnAtoms, n_total, feat, nbr,
                            tile, queue_d, queue_j, rowbuf);
    else if (MANY)
        centroid_group(xyz, sys_first, b * kGroup, n_sys, feat, tile);
    else
        centroid_rows(xyz, sys_first[b], sys_first[b + 1], feat, tile);
}

// ------------------------------------------------------------------ GEMM
// C[m][n] = sum_k A(m, k) B(k, n) with A(m, k) = A[m*sa0 + k*sa1] and
// B(k, n) = B[k*sb0 + n*sb1] (BF16), FP32 accumulation on the matrix cores
// (v_mfma_f32_16x16x16_bf16: lane l holds row l%16 / column l%16 and k =
// 4*(l/16)+q of its A / B fragment, rows 4*(l/16)+q of column l%16 of D).
// Epilogue: + bias[n] (FP32, optional), ReLU (optional), FP32 result to C
// (optional) and its BF16 rounding to Cb (optional).  One wavefront per
// 16x16 tile of C and per slice [y*kc, (y+1)*kc) of k (blockIdx.y = y);
// out-of-range rows, columns and k read as zero.  With several slices
// (P != null) each wave stores its raw FP32 sums to P[y][m][n] and
// k_splitk_reduce adds the slices in order and applies the epilogue, so the
// result does not depend on timing.
typedef short bf16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

__global__ void __launch_bounds__(256) k_gemm(int m, int n, int kdim, int kc, const uint16_t* __restrict__ A,
                                              long sa0, long sa1, const uint16_t* __restrict__ B, long sb0,
                                              long sb1, const float* __restrict__ bias, int relu,
                                              float* __restrict__ C, long ldc, uint16_t* __restrict__ Cb,
                                              long ldcb, float* __restrict__ P) {
    const int wave = threadIdx.x >> 6, l = threadIdx.x & 63;
    const int tiles_n = (n + 15) / 16;
    const long tile = (long)blockIdx.x * 4 + wave;
    const int tm = (int)(tile / tiles_n), tn = (int)(tile % tiles_n);
    if ((long)tm * 16 >= m) return;
    const int row = tm * 16 + (l & 15), col = tn * 16 + (l & 15), kq = 4 * (l >> 4);
    const int k_lo = blockIdx.y * kc, k_hi = min(kdim, k_lo + kc);
    f32x4_t acc = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int k0 = k_lo; k0 < k_hi; k0 += 16) {
        bf16x4_t av, bv;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = k0 + kq + q;
            av[q] = (row < m && k < k_hi) ? (short)A[row * sa0 + k * sa1] : (short)0;
            bv[q] = (col < n && k < k_hi) ? (short)B[k * sb0 + col * sb1] : (short)0;
        }
        acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(av, bv, acc, 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int r = tm * 16 + kq + q;
        if (r >= m || col >= n) continue;
        float v = acc[q];
        if (P) {
            P[((long)blockIdx.y * m + r) * n + col] = v;
            continue;
        }
        if (bias) v += bias[col];
        if (relu) v = fmaxf(v, 0.0f);
        if (C) C[r * ldc + col] = v;
        if (Cb) Cb[r * ldcb + col] = to_bf16(v);
    }
}

__global__ void k_splitk_reduce(int m, int n, int slices, const float* __restrict__ P,
                                const float* __restrict__ bias, int relu, float* __restrict__ C, long ldc,
                                uint16_t* __restrict__ Cb, long ldcb) {
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (long)m * n) return;
    const int r = (int)(e / n), col = (int)(e - (long)r * n);
    float v = 0.0f;
    for (int y = 0; y < slices; ++y) v += P[(long)y * m * n + e];
    if (bias) v += bias[col];
    if (relu) v = fmaxf(v, 0.0f);
    if (C) C[r * ldc + col] = v;
    if (Cb) Cb[r * ldcb + col] = to_bf16(v);
}

// Scratch for the k slices of a product with few output tiles and a long k
// (the weight gradients): at most kMaxSlices slices of a 128 x 128 result.
constexpr int kMaxSlices = 64;
constexpr long kSplitFloats = (long)kMaxSlices * FF_LEARN_HIDDEN * FF_LEARN_HIDDEN;

// LDS-tiled product for operands whose elements run contiguously along k
// or along the other index (every product of the network): a workgroup
// computes a 64 x 64 block of C from 64 x 32 tiles of A and 32 x 64 tiles of
// B staged in LDS with 16-byte loads, each of its four wavefronts a 32 x 32
// quarter (2 x 2 matrix-core tiles) reading 8-byte fragments.  Both tiles are
// kept k-contiguous in LDS: element (r, k) at r * kLdk + k, rows padded to 40
// values so that the 16 rows a fragment read touches fall on different banks.
// A_K: A(i, k) = A[i * sa + k], else A[k * sa + i]; B_K: B(k, j) = B[j * sb + k],
// else B[k * sb + j].  Out-of-range elements load as zero.  k slices, the
// epilogue and the partial sums P as in k_gemm; kc is a multiple of 32.
constexpr int kGbm = 64, kGbn = 64, kGbk = 32, kLdk = kGbk + 8;

template <bool KCONT>
__device__ __forceinline__ void stage_tile(const uint16_t* __restrict__ g, long st, int r0, int r_end, int k0,
                                           int k_end, bool vec_ok, uint16_t* __restrict__ lds) {
    const int t = threadIdx.x;
    uint16_t v[8];
    if (KCONT) {
        // 64 rows x 32 k: thread t loads k [seg, seg + 8) of row t / 4
        const int r = t >> 2, seg = (t & 3) * 8;
        const int row = r0 + r, k = k0 + seg;
        if (vec_ok && row < r_end && k + 8 <= k_end) {
            *(uint4*)v = *(const uint4*)(g + row * st + k);
        } else {
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = (row < r_end && k + q < k_end) ? g[row * st + k + q] : (uint16_t)0;
        }
        *(uint4*)(lds + r * kLdk + seg) = *(const uint4*)v;
    } else {
        // 32 k x 64 rows: thread t loads rows [seg, seg + 8) of k = t / 8
        const int kk = t >> 3, seg = (t & 7) * 8;
        const int k = k0 + kk, row = r0 + seg;
        if (vec_ok && k < k_end && row + 8 <= r_end) {
            *(uint4*)v = *(const uint4*)(g + k * st + row);
        } else {
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = (k < k_end && row + q < r_end) ? g[k * st + row + q] : (uint16_t)0;
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) lds[(seg + q) * kLdk + kk] = v[q];
    }
}

template <bool A_K, bool B_K>
__global__ void __launch_bounds__(256) k_gemm_lds(int m, int n, int kdim, int kc, const uint16_t* __restrict__ A,
                                                  long sa, const uint16_t* __restrict__ B, long sb, int vec_ok,
                                                  const float* __restrict__ bias, int relu, float* __restrict__ C,
                                                  long ldc, uint16_t* __restrict__ Cb, long ldcb,
                                                  float* __restrict__ P) {
    __shared__ __attribute__((aligned(16))) uint16_t As[kGbm * kLdk];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[kGbn * kLdk];
    const int tiles_n = (n + kGbn - 1) / kGbn;
    const int m0 = (int)(blockIdx.x / tiles_n) * kGbm, n0 = (int)(blockIdx.x % tiles_n) * kGbn;
    const int k_lo = blockIdx.y * kc, k_hi = min(kdim, k_lo + kc);
    const int wave = threadIdx.x >> 6, l = threadIdx.x & 63;
    const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    const int fr = l & 15, fk = 4 * (l >> 4);
    f32x4_t acc[2][2] = {};
    for (int k0 = k_lo; k0 < k_hi; k0 += kGbk) {
        stage_tile<A_K>(A, sa, m0, m, k0, k_hi, vec_ok, As);
        stage_tile<B_K>(B, sb, n0, n, k0, k_hi, vec_ok, Bs);
        __syncthreads();
#pragma unroll
        for (int ks = 0; ks < kGbk; ks += 16) {
            bf16x4_t af[2], bf[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                af[u] = *(const bf16x4_t*)(As + (wm + 16 * u + fr) * kLdk + ks + fk);
                bf[u] = *(const bf16x4_t*)(Bs + (wn + 16 * u + fr) * kLdk + ks + fk);
            }
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int w = 0; w < 2; ++w)
                    acc[u][w] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(af[u], bf[w], acc[u][w], 0, 0, 0);
        }
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int w = 0; w < 2; ++w)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int r = m0 + wm + 16 * u + fk + q, col = n0 + wn + 16 * w + fr;
                if (r >= m || col >= n) continue;
                float v = acc[u][w][q];
                if (P) {
                    P[((long)blockIdx.y * m + r) * n + col] = v;
                    continue;
                }
                if (bias) v += bias[col];
                if (relu) v = fmaxf(v, 0.0f);
                if (C) C[r * ldc + col] = v;
                if (Cb) Cb[r * ldcb + col] = to_bf16(v);
            }
}

hipError_t launch_gemm(int m, int n, int k, const uint16_t* A, long sa0, long sa1, const uint16_t* B, long sb0,
                       long sb1, const float* bias, int relu, float* C, long ldc, uint16_t* Cb, long ldcb,
                       hipStream_t s, float* split = nullptr, long split_floats = 0) {
    // the tiled kernel takes operands contiguous along one index, blocks of
    // at least 64 x 64 x 32; 16-byte loads where strides and bases allow
    const bool a_k = sa1 == 1, a_m = sa0 == 1 && !a_k, b_k = sb0 == 1, b_n = sb1 == 1 && !b_k;
    const bool tiled = (a_k || a_m) && (b_k || b_n) && m >= kGbm && n >= kGbn && k >= kGbk;
    const long blocks = tiled ? (long)((m + kGbm - 1) / kGbm) * ((n + kGbn - 1) / kGbn)
                              : ((long)((m + 15) / 16) * ((n + 15) / 16) + 3) / 4;
    int slices = 1;
    // split k when the output blocks alone cannot fill the chip: slices of >= 256
    if (split && blocks < 256 && k >= 512) {
        const long by_k = k / 256, by_ws = split_floats / ((long)m * n);
        slices = (int)std::max(1L, std::min({by_k, by_ws, (long)kMaxSlices}));
    }
    const int step = tiled ? kGbk : 16;
    const int kc = slices == 1 ? k : ((k + slices - 1) / slices + step - 1) / step * step;
    slices = (k + kc - 1) / kc;
    float* P = slices > 1 ? split : nullptr;
    if (tiled) {
        const long sa = a_k ? sa0 : sa1, sb = b_k ? sb1 : sb0;
        const int vec = ((uintptr_t)A % 16 == 0) && ((uintptr_t)B % 16 == 0) && sa % 8 == 0 && sb % 8 == 0;
        const dim3 grid((unsigned)blocks, (unsigned)slices);
        if (a_k && b_k)
            hipLaunchKernelGGL((k_gemm_lds<true, true>), grid, dim3(256), 0, s, m, n, k, kc, A, sa, B, sb, vec, bias,
                               relu, C, ldc, Cb, ldcb, P);
        else if (a_k)
            hipLaunchKernelGGL((k_gemm_lds<true, false>), grid, dim3(256), 0, s, m, n, k, kc, A, sa, B, sb, vec, bias,
                               relu, C, ldc, Cb, ldcb, P);
        else if (b_k)
            hipLaunchKernelGGL((k_gemm_lds<false, true>), grid, dim3(256), 0, s, m, n, k, kc, A, sa, B, sb, vec, bias,
                               relu, C, ldc, Cb, ldcb, P);
        else
            hipLaunchKernelGGL((k_gemm_lds<false, false>), grid, dim3(256), 0, s, m, n, k, kc, A, sa, B, sb, vec,
                               bias, relu, C, ldc, Cb, ldcb, P);
    } else {
        hipLaunchKernelGGL(k_gemm, dim3((unsigned)blocks, (unsigned)slices), dim3(256), 0, s, m, n, k, kc, A, sa0, sa1,
                           B, sb0, sb1, bias, relu, C, ldc, Cb, ldcb, P);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !P) return e;
    const long mn = (long)m * n;
    hipLaunchKernelGGL(k_splitk_reduce, dim3((unsigned)((mn + 255) / 256)), dim3(256), 0, s, m, n, slices, P, bias,
                       relu, C, ldc, Cb, ldcb);
    return hipGetLastError();
}

// ------------------------------------------------------------------ network
// Parameter offsets (elements) in the packed vector.
constexpr long kW1 = 0, kB1 = kW1 + (long)FF_LEARN_FEATURES * FF_LEARN_HIDDEN;
constexpr long kW2 = kB1 + FF_LEARN_HIDDEN, kB2 = kW2 + (long)FF_LEARN_HIDDEN * FF_LEARN_HIDDEN;
constexpr long kW3 = kB2 + FF_LEARN_HIDDEN, kB3 = kW3 + (long)FF_LEARN_HIDDEN * FF_LEARN_OUT_PAD;
constexpr long kParams = kB3 + FF_LEARN_OUT_PAD;
static_assert(FF_LEARN_FEATURES == 128 && FF_LEARN_HIDDEN == 128 && FF_LEARN_OUT_PAD == 16,
              "fragment counts of the fused network");

// The three layers of 16 rows run in the registers of one wavefront.  The
// matrix-core fragments of both operands hold index l % 16 and k = 4 (l / 16) + q
// in lane l, and a product comes back with its second operand's index at l % 16
// and the first's at 4 (l / 16) + q.  So with the weights as the first operand
// (and the rows as the second) the activations of one layer, rounded to BF16,
// are the operand of the next; with the operands exchanged they come back with
// the roles of row and column exchanged, which is what the weight gradients
// contract over.  k runs in the same order as in k_gemm.
constexpr int kT = 8;                        // 16-wide tiles of a 128-wide layer
constexpr int kLdw = 128 + 8;                // weights in LDS: [output][input], padded against bank conflicts
constexpr int kRowBlock = 64;                // rows of a workgroup at a time: 16 per wavefront

typedef __bf16 hwbf16x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ bf16x4_t pack_bf16(const f32x4_t& v) {          // v_cvt_pk_bf16_f32: nearest even
    return __builtin_bit_cast(bf16x4_t, __builtin_convertvector(v, hwbf16x4_t));
}
__device__ __forceinline__ f32x4_t mfma16(const bf16x4_t& a, const bf16x4_t& b, const f32x4_t& c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// W [128][COLS] (row-major, BF16) through registers into LDS as [COLS][kLdw]
// (store) and, where wanted, also as it is with rows of kLdw (store_rows).  A
// thread takes 4 x 4 elements at a time; the 8 x 8 pattern of a wavefront keeps
// the writes free of bank conflicts.  The loads of all weights are issued
// before the first store: one memory latency, not one for each.
template <int COLS>
struct StagedWeights {
    static constexpr int kTasks = 32 * (COLS / 4);
    static constexpr int kPer = (kTasks + 255) / 256;
    uint2 w[kPer][4];
    __device__ __forceinline__ static int column(int task) {
        return COLS == 128 ? 4 * (((task >> 6) & 3) * 8 + (task & 7)) : 4 * (task & 3);
    }
    __device__ __forceinline__ static int row(int task) {
        return COLS == 128 ? 4 * ((task >> 8) * 8 + ((task >> 3) & 7)) : 4 * ((task >> 2) & 31);
    }
    __device__ __forceinline__ void load(const uint16_t* __restrict__ W) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int task = threadIdx.x + 256 * i;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (task < kTasks) w[i][q] = *(const uint2*)(W + (row(task) + q) * COLS + column(task));
        }
    }
    __device__ __forceinline__ void store(uint16_t* __restrict__ lds) const {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int task = threadIdx.x + 256 * i;
            if (task >= kTasks) continue;
            uint16_t* p = lds + column(task) * kLdw + row(task);
            const uint2(&v)[4] = w[i];
            *(uint2*)(p) = make_uint2((v[0].x & 0xffffu) | (v[1].x << 16), (v[2].x & 0xffffu) | (v[3].x << 16));
            *(uint2*)(p + kLdw) = make_uint2((v[0].x >> 16) | (v[1].x & 0xffff0000u), (v[2].x >> 16) | (v[3].x & 0xffff0000u));
            *(uint2*)(p + 2 * kLdw) = make_uint2((v[0].y & 0xffffu) | (v[1].y << 16), (v[2].y & 0xffffu) | (v[3].y << 16));
            *(uint2*)(p + 3 * kLdw) = make_uint2((v[0].y >> 16) | (v[1].y & 0xffff0000u), (v[2].y >> 16) | (v[3].y & 0xffff0000u));
        }
    }
    __device__ __forceinline__ void store_rows(uint16_t* __restrict__ lds) const {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int task = threadIdx.x + 256 * i;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (task < kTasks) *(uint2*)(lds + (row(task) + q) * kLdw + column(task)) = w[i][q];
        }
    }
};
// Fragment of the staged weights: output tile nt, input tile kt.
__device__ __forceinline__ bf16x4_t weight_frag(const uint16_t* lds, int nt, int kt, int l) {
    return *(const bf16x4_t*)(lds + (nt * 16 + (l & 15)) * kLdw + kt * 16 + 4 * (l >> 4));
}

// Bias, ReLU and BF16 of one tile; the bits of the positive values go to
// positive[4 t ..].
__device__ __forceinline__ bf16x4_t relu_tile(f32x4_t acc, const f32x4_t& b, int t, uint32_t& positive) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        acc[q] = fmaxf(acc[q] + b[q], 0.0f);
        if (acc[q] > 0.0f) positive |= 1u << (4 * t + q);
    }
    return pack_bf16(acc);
}
// A hidden layer of the wavefront's rows.  `out`: the next layer's operand (the
// lane's row at l % 16).  BOTH: also with the operands exchanged, `by_rows`
// (rows 4 (l / 16) + q at unit l % 16 of each tile); both from one read of the
// weights.  The masks hold the positive activations.
template <bool BOTH>
__device__ __forceinline__ void hidden_layer(const uint16_t* w, const float* __restrict__ bias, const bf16x4_t (&in)[kT],
                                             int l, bf16x4_t (&out)[kT], uint32_t& positive, bf16x4_t (&by_rows)[kT],
                                             uint32_t& positive_rows) {
    positive = positive_rows = 0;
#pragma unroll
    for (int n0 = 0; n0 < kT; n0 += 4) {
        f32x4_t acc[4] = {}, acr[4] = {};
#pragma unroll
        for (int kt = 0; kt < kT; ++kt)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const bf16x4_t f = weight_frag(w, n0 + u, kt, l);
                acc[u] = mfma16(f, in[kt], acc[u]);
                if (BOTH) acr[u] = mfma16(in[kt], f, acr[u]);
            }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int t = n0 + u;
            out[t] = relu_tile(acc[u], *(const f32x4_t*)(bias + t * 16 + 4 * (l >> 4)), t, positive);
            if (BOTH) {
                const float b = bias[t * 16 + (l & 15)];
                by_rows[t] = relu_tile(acr[u], f32x4_t{b, b, b, b}, t, positive_rows);
            }
        }
    }
}
__device__ __forceinline__ void load_biases(const float* __restrict__ params, float* bias) {
    for (int k = threadIdx.x; k < 272; k += 256)
        bias[k] = params[k < 128 ? kB1 + k : (k < 256 ? kB2 + k - 128 : kB3 + k - 256)];
}

// BF16 feature fragments of row `row` (zeros past the end).
__device__ __forceinline__ void load_rows(const uint16_t* __restrict__ X, int row, int n, int l, bf16x4_t (&x)[kT]) {
    const uint16_t* p = X + (size_t)min(row, n - 1) * FF_LEARN_FEATURES + 4 * (l >> 4);
#pragma unroll
    for (int kt = 0; kt < kT; ++kt) x[kt] = *(const bf16x4_t*)(p + kt * 16);
    if (row >= n)
#pragma unroll
        for (int kt = 0; kt < kT; ++kt) x[kt] = bf16x4_t{0, 0, 0, 0};
}

// Network output of every row: one launch, weights staged once per workgroup,
// activations in registers.  Bound by latency (weights, then two layers): 7.5 us
// at 10,000 rows; three products with BF16 and FP32 activations in memory
// between them took 32 us.
constexpr int kForwardGrid = 512;            // two workgroups of 74 KB LDS per CU
__global__ void __launch_bounds__(256, 2) k_forward(const float* __restrict__ params, const uint16_t* __restrict__ wb,
                                                 const uint16_t* __restrict__ X, int n, float* __restrict__ Y) {
    __shared__ __attribute__((aligned(16))) uint16_t w1[128 * kLdw], w2[128 * kLdw], w3[16 * kLdw];
    __shared__ __attribute__((aligned(16))) float bias[272];
    const int l = threadIdx.x & 63, wave = threadIdx.x >> 6;
    bf16x4_t x[kT], h1[kT], h2[kT], none[kT];
    load_rows(X, blockIdx.x * kRowBlock + wave * 16 + (l & 15), n, l, x);
    {
        StagedWeights<128> s1, s2;
        StagedWeights<16> s3;
        s1.load(wb + kW1);
        s2.load(wb + kW2);
        s3.load(wb + kW3);
        load_biases(params, bias);
        s1.store(w1);
        s2.store(w2);
        s3.store(w3);
    }
    __syncthreads();
    for (int r0 = blockIdx.x * kRowBlock; r0 < n; r0 += gridDim.x * kRowBlock) {
        // weights are read again for each row block (kept across the loop they
        // would fill the registers)
        asm volatile("" : : : "memory");
        const int row = r0 + wave * 16 + (l & 15);
        uint32_t mask, mask_rows;
        hidden_layer<false>(w1, bias, x, l, h1, mask, none, mask_rows);
        if (r0 + (int)gridDim.x * kRowBlock < n) load_rows(X, row + gridDim.x * kRowBlock, n, l, x);
        hidden_layer<false>(w2, bias + 128, h1, l, h2, mask, none, mask_rows);
        f32x4_t y = {};
#pragma unroll
        for (int kt = 0; kt < kT; ++kt) y = mfma16(weight_frag(w3, 0, kt, l), h2[kt], y);
        y += *(const f32x4_t*)(bias + 256 + 4 * (l >> 4));
        if (row < n) *(f32x4_t*)(Y + (size_t)row * FF_LEARN_OUT_PAD + 4 * (l >> 4)) = y;
    }
}

// Forward and backward pass of one minibatch up to per-workgroup partial sums
// of the gradient: one launch, then k_gradient_sum.  A wavefront computes the
// activations and their gradients of its 16 rows in registers, in both
// orientations (see above): the one with the lane's row at l % 16 feeds the next
// product, the other one (rows at 4 (l / 16) + q) goes to LDS as a fragment.
// Then wavefront w forms the weight gradients of input tiles 2w and 2w + 1 over
// the workgroup's 64 rows, which stay in its registers over all of its row
// blocks.  Bias gradients and the loss are summed in FP64.
// 8,192 rows: 26 us and 5.6 us for the sum, of which 4.5 us stage the weights,
// 10 us are products and 3.6 us the store of the partials (18 MB); 15 launches
// with every activation and gradient in memory in FP32 and BF16 took 150 us.
constexpr int kTrainGrid = 256;              // one workgroup of 159 KB LDS per CU
constexpr int kBiasSums = 128 + 128 + 16 + 1;         // FP64 partials of a workgroup: db1, db2, db3, loss
constexpr size_t kTrainPartial = ((size_t)kParams * 4 + kBiasSums * 8 + 255) / 256 * 256;   // bytes per workgroup

__global__ void __launch_bounds__(256, 1) k_train_block(const float* __restrict__ params,
                                                        const uint16_t* __restrict__ wb,
                                                        const uint16_t* __restrict__ X, int n,
                                                        const float* __restrict__ target, char* __restrict__ partial) {
    __shared__ __attribute__((aligned(16))) uint16_t w1[128 * kLdw], w2[128 * kLdw], w3[16 * kLdw];
    __shared__ __attribute__((aligned(16))) uint16_t w2r[128 * kLdw];       // W2 itself, [input][output]
    __shared__ __attribute__((aligned(16))) float bias[272];
    // fragments of the workgroup's row groups, [group][tile][lane]
    __shared__ bf16x4_t frag[3][4][kT][64];
    auto f_h1 = frag[0], f_d2 = frag[1], f_d1 = frag[2];
    const int l = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lc = l & 15, lr = 4 * (l >> 4);
    bf16x4_t x[kT];
    load_rows(X, blockIdx.x * kRowBlock + wave * 16 + lc, n, l, x);
    bf16x4_t w3r[kT];                        // W3 rows: hidden unit l % 16 of each tile, outputs lr ..
#pragma unroll
    for (int t = 0; t < kT; ++t) w3r[t] = *(const bf16x4_t*)(wb + kW3 + (t * 16 + lc) * FF_LEARN_OUT_PAD + lr);
    {
        StagedWeights<128> s1, s2;
        StagedWeights<16> s3;
        s1.load(wb + kW1);
        s2.load(wb + kW2);
        s3.load(wb + kW3);
        load_biases(params, bias);
        s1.store(w1);
        s2.store(w2);
        s2.store_rows(w2r);
        s3.store(w3);
    }
    __syncthreads();
    f32x4_t dw1[2][kT] = {}, dw2[2][kT] = {}, dw3[kT] = {};
    double db1[kT] = {}, db2[kT] = {}, db3 = 0.0, loss = 0.0;
    const float inv = 3.0f * (float)n;
    for (int r0 = blockIdx.x * kRowBlock; r0 < n; r0 += gridDim.x * kRowBlock) {
        // weights are read again for each row block (kept across the loop they
        // would fill the registers)
        asm volatile("" : : : "memory");
        const int rw = r0 + wave * 16;       // the wavefront's first row
        // features by rows for dW1, and the targets: used later, loaded now
        bf16x4_t xr[4][2];
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int row = r0 + g * 16 + lr + q;
                    const short v = (short)X[(size_t)min(row, n - 1) * FF_LEARN_FEATURES + (2 * wave + u) * 16 + lc];
                    xr[g][u][q] = row < n ? v : (short)0;
                }
        float tg[3], tgr[4];
#pragma unroll
        for (int c = 0; c < 3; ++c) tg[c] = target[3 * (size_t)min(rw + lc, n - 1) + c];
#pragma unroll
        for (int q = 0; q < 4; ++q) tgr[q] = target[3 * (size_t)min(rw + lr + q, n - 1) + min(lc, 2)];
        {
            bf16x4_t h[kT], h2[kT], hr[kT];
            uint32_t p1, p1r, p2, p2r;
            hidden_layer<true>(w1, bias, x, l, h, p1, hr, p1r);
#pragma unroll
            for (int t = 0; t < kT; ++t) f_h1[wave][t][l] = hr[t];
            if (r0 + (int)gridDim.x * kRowBlock < n) load_rows(X, rw + lc + gridDim.x * kRowBlock, n, l, x);
            hidden_layer<true>(w2, bias + 128, h, l, h2, p2, hr, p2r);
            // output, its error and gradient dY = 2 (Y - T) / (3 n) on the three
            // used columns, both ways
            f32x4_t y = {}, yr = {};
#pragma unroll
            for (int kt = 0; kt < kT; ++kt) {
                const bf16x4_t w = weight_frag(w3, 0, kt, l);
                y = mfma16(w, h2[kt], y);
                yr = mfma16(h2[kt], w, yr);
            }
            f32x4_t dy = {}, dyr = {};
            if (l < 16 && rw + lc < n)
#pragma unroll
                for (int c = 0; c < 3; ++c) dy[c] = 2.0f * (y[c] + bias[256 + c] - tg[c]) / inv;
            if (lc < 3)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (rw + lr + q < n) {
                        const float e = yr[q] + bias[256 + lc] - tgr[q];
                        dyr[q] = 2.0f * e / inv;
                        loss += (double)(e * e);
                        db3 += (double)dyr[q];
                    }
            const bf16x4_t fdy = pack_bf16(dy), fdyr = pack_bf16(dyr);
            // dW3 += H2^T dY over the wavefront's rows; dH2 = dY W3^T where H2 > 0
            bf16x4_t d2[kT];
#pragma unroll
            for (int t = 0; t < kT; ++t) {
                dw3[t] = mfma16(hr[t], fdyr, dw3[t]);
                f32x4_t a = mfma16(w3r[t], fdy, f32x4_t{}), ar = mfma16(fdy, w3r[t], f32x4_t{});
                double s = 0.0;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    a[q] = (p2 >> (4 * t + q)) & 1u ? a[q] : 0.0f;
                    ar[q] = (p2r >> (4 * t + q)) & 1u ? ar[q] : 0.0f;
                    s += (double)ar[q];
                }
                db2[t] += s;
                d2[t] = pack_bf16(a);
                f_d2[wave][t][l] = pack_bf16(ar);
            }
            // dH1 = dH2 W2^T where H1 > 0 (by rows only)
#pragma unroll
            for (int t0 = 0; t0 < kT; t0 += 4) {
                f32x4_t ar[4] = {};
#pragma unroll
                for (int kt = 0; kt < kT; ++kt)
#pragma unroll
                    for (int u = 0; u < 4; ++u) ar[u] = mfma16(d2[kt], weight_frag(w2r, t0 + u, kt, l), ar[u]);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int t = t0 + u;
                    double s = 0.0;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        ar[u][q] = (p1r >> (4 * t + q)) & 1u ? ar[u][q] : 0.0f;
                        s += (double)ar[u][q];
                    }
                    db1[t] += s;
                    f_d1[wave][t][l] = pack_bf16(ar[u]);
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const bf16x4_t h1[2] = {f_h1[g][2 * wave][l], f_h1[g][2 * wave + 1][l]};
#pragma unroll
            for (int t = 0; t < kT; ++t) {
                const bf16x4_t d2 = f_d2[g][t][l], d1 = f_d1[g][t][l];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    dw2[u][t] = mfma16(h1[u], d2, dw2[u][t]);
                    dw1[u][t] = mfma16(xr[g][u], d1, dw1[u][t]);
                }
            }
        }
        __syncthreads();
    }
    float* out = (float*)(partial + blockIdx.x * kTrainPartial);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int m = (2 * wave + u) * 16 + lr + q;
#pragma unroll
            for (int t = 0; t < kT; ++t) {
                out[kW1 + m * FF_LEARN_HIDDEN + t * 16 + lc] = dw1[u][t][q];
                out[kW2 + m * FF_LEARN_HIDDEN + t * 16 + lc] = dw2[u][t][q];
            }
        }
    // dW3: the wavefronts' sums through the fragments' LDS, added in order
    static_assert(sizeof frag >= 4 * 2048 * 4, "dW3 of four wavefronts");
    float* s3 = (float*)frag;
#pragma unroll
    for (int t = 0; t < kT; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) s3[wave * 2048 + (t * 16 + lr + q) * FF_LEARN_OUT_PAD + lc] = dw3[t][q];
    // column sums: over the lanes that share a column, then the wavefronts
    // (through the weights' LDS, which is no longer needed)
    double* sums = (double*)w1;
    auto fold = [&](double v) {
        v += __shfl_xor(v, 16, 64);
        return v + __shfl_xor(v, 32, 64);
    };
    __syncthreads();
#pragma unroll
    for (int t = 0; t < kT; ++t) {
        const double a = fold(db1[t]), b = fold(db2[t]);
        if (l < 16) {
            sums[wave * kBiasSums + t * 16 + l] = a;
            sums[wave * kBiasSums + 128 + t * 16 + l] = b;
        }
    }
    const double c = fold(db3);
    double e = fold(loss);
    e += __shfl_xor(e, 1, 64) + __shfl_xor(e, 2, 64);      // lane 0: columns 0, 1, 2
    if (l < 16) sums[wave * kBiasSums + 256 + l] = c;
    if (l == 0) sums[wave * kBiasSums + 272] = e;
    __syncthreads();
    for (int k = threadIdx.x; k < 2048; k += 256)
        out[kW3 + k] = (s3[k] + s3[2048 + k]) + (s3[4096 + k] + s3[6144 + k]);
    double* dbias = (double*)(out + kParams);
    static_assert(kParams % 2 == 0, "FP64 partials behind the FP32 ones");
    for (int k = threadIdx.x; k < kBiasSums; k += 256)
        dbias[k] = (sums[k] + sums[kBiasSums + k]) + (sums[2 * kBiasSums + k] + sums[3 * kBiasSums + k]);
}

// Gradient and loss from the workgroups' partial sums, added in FP64 in a fixed
// order.  A workgroup takes 128 entries: eight groups of 32 threads take four
// entries each (16-byte loads) of an eighth of the partials.  The entries of a
// workgroup are all weights (FP32 partials) or all biases (FP64; the last
// workgroup's: b3 and the loss).
constexpr int kSumEntries = 128;
static_assert(kB1 % kSumEntries == 0 && kW2 % kSumEntries == 0 && kB2 % kSumEntries == 0 && kW3 % kSumEntries == 0 &&
              kB3 % kSumEntries == 0, "a workgroup's entries are all weights or all biases");
__global__ void __launch_bounds__(256) k_gradient_sum(const char* __restrict__ partial, int parts, double loss_scale,
                                                      float* __restrict__ grad, float* __restrict__ loss) {
    __shared__ double red[8][kSumEntries];
    const int t = threadIdx.x, sub = t & 31, grp = t >> 5;
    const int e0 = blockIdx.x * kSumEntries;
    const int lo = parts * grp / 8, hi = parts * (grp + 1) / 8;
    // first bias entry of the workgroup, or -1 for weights
    const int b0 = e0 == kB1 ? 0 : (e0 == kB2 ? 128 : (e0 == kB3 ? 256 : -1));
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    constexpr int kAhead = 16;               // partials in flight per thread
    for (int p0 = lo; p0 < hi; p0 += kAhead) {
        if (b0 < 0) {
            f32x4_t v[kAhead];
#pragma unroll
            for (int i = 0; i < kAhead; ++i)
                v[i] = *(const f32x4_t*)(partial + min(p0 + i, hi - 1) * kTrainPartial + 4 * (size_t)(e0 + 4 * sub));
#pragma unroll
            for (int i = 0; i < kAhead; ++i)
#pragma unroll
                for (int k = 0; k < 4; ++k) s[k] += p0 + i < hi ? (double)v[i][k] : 0.0;
        } else {
            double v[kAhead][4];
#pragma unroll
            for (int i = 0; i < kAhead; ++i)
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    v[i][k] = ((const double*)(partial + min(p0 + i, hi - 1) * kTrainPartial +
                                               kParams * 4))[min(b0 + 4 * sub + k, kBiasSums - 1)];
#pragma unroll
            for (int i = 0; i < kAhead; ++i)
#pragma unroll
                for (int k = 0; k < 4; ++k) s[k] += p0 + i < hi ? v[i][k] : 0.0;
        }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) red[grp][4 * sub + k] = s[k];
    __syncthreads();
    if (t >= kSumEntries) return;
    double v = red[0][t];
#pragma unroll
    for (int k = 1; k < 8; ++k) v += red[k][t];
    if (e0 + t < kParams) grad[e0 + t] = (float)v;
    else if (e0 + t == kParams) *loss = (float)(loss_scale * v);
}

// ------------------------------------------------------ loss and backward
// dY = 2 (Y - T) / (3 n) over the 3 used outputs (zero in the padding), as
// FP32 and BF16; per-row squared errors for the loss.
__global__ void k_mse(int n, const float* __restrict__ Y, const float* __restrict__ T, float* __restrict__ dY,
                      uint16_t* __restrict__ dYb, float* __restrict__ row_loss) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float l = 0.0f;
    for (int c = 0; c < FF_LEARN_OUT_PAD; ++c) {
        float d = 0.0f;
        if (c < 3) {
            const float e = Y[(size_t)i * FF_LEARN_OUT_PAD + c] - T[3 * (size_t)i + c];
            l += e * e;
            d = 2.0f * e / (3.0f * (float)n);
        }
        dY[(size_t)i * FF_LEARN_OUT_PAD + c] = d;
        dYb[(size_t)i * FF_LEARN_OUT_PAD + c] = to_bf16(d);
    }
    row_loss[i] = l;
}

// dH = dH * (H > 0), then its BF16 copy.
__global__ void k_relu_back(long count, const float* __restrict__ H, float* __restrict__ dH,
                            uint16_t* __restrict__ dHb) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    const float v = H[i] > 0.0f ? dH[i] : 0.0f;
    dH[i] = v;
    dHb[i] = to_bf16(v);
}

// out[c] = scale * sum_i X[i][c] for an FP32 [n][cols] matrix (bias
// gradients, and the loss from per-row errors).  One block per column; each
// thread sums a fixed stride of rows in FP64, then a fixed-order tree, so the
// result does not depend on timing.
__global__ void __launch_bounds__(256) k_colsum(int n, int cols, const float* __restrict__ X, double scale,
                                                float* __restrict__ out) {
    __shared__ double red[256];
    const int c = blockIdx.x;
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) s += X[(size_t)i * cols + c];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[c] = (float)(scale * red[0]);
}

// ------------------------------------------------------------------ Adam
__global__ void k_adam(int count, float* __restrict__ w, uint16_t* __restrict__ wb, const float* __restrict__ g,
                       float* __restrict__ m, float* __restrict__ v, float lr, float b1, float b2, float eps,
                       float c1, float c2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float wi = w[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    w[i] = wi;
    if (wb) wb[i] = to_bf16(wi);
}

// ------------------------------------------------------------- apply
// x_out = x_in + scale * disp (FP32 displacement [n][3], padded rows of
// FF_LEARN_OUT_PAD), FP64 points.
__global__ void k_displace(long n3, const double* __restrict__ x, const float* __restrict__ disp, double scale,
                           double* __restrict__ out) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n3) return;
    const long a = i / 3, c = i - 3 * a;
    out[i] = x[i] + scale * (double)disp[a * FF_LEARN_OUT_PAD + c];
}

__global__ void k_to_bf16(long n, const float* __restrict__ x, uint16_t* __restrict__ out) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = to_bf16(x[i]);
}

__global__ void k_delta(long n3, const double* __restrict__ a, const double* __restrict__ b, float* __restrict__ out) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n3) out[i] = (float)(b[i] - a[i]);
}

__device__ __forceinline__ bool take_new(double e_old, double e_new) {
    return e_new < e_old && e_new - e_new == 0.0;   // finite and lower
}

// out may alias x_old (each element is read and written by one thread)
__global__ void k_select(long n3, const double* x_old, const double* __restrict__ x_new,
                         const double* __restrict__ e_old, const double* __restrict__ e_new,
                         const int32_t* __restrict__ atom_sys, double* out) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n3) return;
    const int s = atom_sys[i / 3];
    out[i] = take_new(e_old[s], e_new[s]) ? x_new[i] : x_old[i];
}

// runs after k_select (same stream), so e_out may alias e_old
__global__ void k_chosen(int n_sys, const double* e_old, const double* __restrict__ e_new, int32_t* chosen,
                         double* e_out) {
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n_sys) return;
    const bool t = take_new(e_old[s], e_new[s]);
    if (chosen) chosen[s] = t ? 1 : 0;
    if (e_out) e_out[s] = t ? e_new[s] : e_old[s];
}

__global__ void k_gather(const uint32_t* __restrict__ src, const int32_t* __restrict__ idx, long n_rows,
                         int words, uint32_t* __restrict__ dst) {
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n_rows * words) return;
    const long r = t / words, w = t - r * words;
    dst[t] = src[(long)idx[r] * words + w];
}

}  // namespace ff

// =================================================================== C ABI
using namespace ff;

namespace {
thread_local std::string g_learn_err;
ff_status lfail(ff_status st, const char* fmt, ...) {
    char buf[256];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_learn_err = buf;
    return st;
}
#define L_TRY(expr)                                                                             \
    do {                                                                                        \
        hipError_t e_ = (expr);                                                                 \
        if (e_ != hipSuccess) return lfail(FF_ERR_HIP, "%s: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

// activation workspace (bytes) for n rows
size_t act_bytes(long n) {
    const long h = FF_LEARN_HIDDEN, o = FF_LEARN_OUT_PAD;
    return (size_t)n * (2 * h * 4 + 2 * h * 2 + o * 4) + 256 * 8;
}
// The fused network reads features and weights 8 bytes at a time; arrays that
// are aligned to less take the products one by one.
bool fused_ok(const uint16_t* features, const uint16_t* params_bf16) {
    return (uintptr_t)features % 8 == 0 && (uintptr_t)params_bf16 % 8 == 0;
}
struct Act {
    float *h1, *h2, *y;
    uint16_t *h1b, *h2b;
};
Act carve(void* ws, long n) {
    char* p = (char*)ws;
    auto take = [&](size_t b) { char* r = p; p += (b + 255) & ~(size_t)255; return r; };
    const long h = FF_LEARN_HIDDEN;
    Act a;
    a.h1 = (float*)take((size_t)n * h * 4);
    a.h2 = (float*)take((size_t)n * h * 4);
    a.h1b = (uint16_t*)take((size_t)n * h * 2);
    a.h2b = (uint16_t*)take((size_t)n * h * 2);
    a.y = (float*)take((size_t)n * FF_LEARN_OUT_PAD * 4);
    return a;
}
}  // namespace

extern "C" {

int32_t ff_learn_param_count(void) { return (int32_t)kParams; }

// forward: the activations; backward: activations, their gradients and the
// k-slice scratch of the weight gradients
size_t backward_bytes(long n) { return 2 * act_bytes(n) + (size_t)kSplitFloats * 4; }

size_t ff_learn_workspace_bytes(int32_t n_rows) { return n_rows < 1 ? 0 : backward_bytes(n_rows) + 2 * 256; }

const char* ff_learn_last_error(void) { return g_learn_err.c_str(); }

ff_status ff_learn_features(int32_t n_sys, int32_t n_total, const double* xyz, const double* q,
                            const double* sigma, const double* eps, const int32_t* sys_first,
                            const int32_t* atom_sys, uint16_t* features, int32_t* neighbors, void* stream) {
    g_learn_err.clear();
    if (n_sys < 1 || n_total < 1) return lfail(FF_ERR_ARG, "need at least one system and one atom");
    if (!xyz || !q || !sigma || !eps || !sys_first || !atom_sys || !features) return lfail(FF_ERR_ARG, "null pointer");
    // many small systems are more centroid workgroups than the chip holds at a
    // time beside the others (five a CU): 3,000 systems of three atoms take
    // 18.6 us with a workgroup each, 10.0 in groups; 64 of 63 atoms 11.8 and 14.1
    const bool many = n_sys >= 640 && n_total <= 16LL * n_sys;
    const int blocks = (many ? (n_sys + kGroup - 1) / kGroup : n_sys) + (n_total + 4 * kKnnAtoms - 1) / (4 * kKnnAtoms);
    hipLaunchKernelGGL(many ? k_features<true> : k_features<false>, dim3(blocks), dim3(256), 0, (hipStream_t)stream, xyz,
                       q, sigma, eps, sys_first, atom_sys, n_sys, n_total, features, neighbors);
    L_TRY(hipGetLastError());
    return FF_OK;
}

ff_status ff_learn_gemm(int32_t m, int32_t n, int32_t k, const uint16_t* a, int64_t sa0, int64_t sa1,
                        const uint16_t* b, int64_t sb0, int64_t sb1, const float* bias, int32_t relu, float* c,
                        int64_t ldc, uint16_t* cb, int64_t ldcb, void* stream) {
    g_learn_err.clear();
    if (m < 1 || n < 1 || k < 1 || !a || !b || (!c && !cb)) return lfail(FF_ERR_ARG, "bad GEMM arguments");
    L_TRY(launch_gemm(m, n, k, a, sa0, sa1, b, sb0, sb1, bias, relu, c, ldc, cb, ldcb, (hipStream_t)stream));
    return FF_OK;
}

ff_status ff_learn_forward(const float* params, const uint16_t* params_bf16, const uint16_t* features,
                           int32_t n_rows, void* workspace, size_t workspace_bytes, float* out, void* stream) {
    g_learn_err.clear();
    if (!params || !params_bf16 || !features || n_rows < 1 || !workspace || !out)
        return lfail(FF_ERR_ARG, "null argument or no rows");
    if (workspace_bytes < act_bytes(n_rows) || ((uintptr_t)workspace & 255))
        return lfail(FF_ERR_WORKSPACE, "workspace too small or misaligned");
    hipStream_t st = (hipStream_t)stream;
    if (fused_ok(features, params_bf16) && (uintptr_t)out % 16 == 0) {
        const int blocks = (n_rows + kRowBlock - 1) / kRowBlock;
        hipLaunchKernelGGL(k_forward, dim3(std::min(blocks, kForwardGrid)), dim3(256), 0, st, params, params_bf16,
                           features, n_rows, out);
        L_TRY(hipGetLastError());
        return FF_OK;
    }
    const Act t = carve(workspace, n_rows);
    const long F = FF_LEARN_FEATURES, H = FF_LEARN_HIDDEN, O = FF_LEARN_OUT_PAD;
    // H1 = relu(X W1 + b1), H2 = relu(H1 W2 + b2), Y = H2 W3 + b3
    L_TRY(launch_gemm(n_rows, H, F, features, F, 1, params_bf16 + kW1, H, 1, params + kB1, 1, t.h1, H, t.h1b, H, st));
    L_TRY(launch_gemm(n_rows, H, H, t.h1b, H, 1, params_bf16 + kW2, H, 1, params + kB2, 1, t.h2, H, t.h2b, H, st));
    L_TRY(launch_gemm(n_rows, O, H, t.h2b, H, 1, params_bf16 + kW3, O, 1, params + kB3, 0, out, O, nullptr, 0, st));
    return FF_OK;
}

ff_status ff_learn_backward(const float* params, const uint16_t* params_bf16, const uint16_t* features,
                            int32_t n_rows, void* workspace, size_t workspace_bytes, const float* target,
                            float* grad, float* loss, void* stream) {
    g_learn_err.clear();
    if (!params || !params_bf16 || !features || n_rows < 1 || !workspace || !target || !grad || !loss)
        return lfail(FF_ERR_ARG, "null argument or no rows");
    const size_t need = backward_bytes(n_rows);
    if (workspace_bytes < need || ((uintptr_t)workspace & 255))
        return lfail(FF_ERR_WORKSPACE, "workspace too small or misaligned (%zu needed)", need);
    hipStream_t st = (hipStream_t)stream;
    if (fused_ok(features, params_bf16)) {
        const int parts = std::min((n_rows + kRowBlock - 1) / kRowBlock, kTrainGrid);
        static_assert(kTrainPartial <= kRowBlock * (2 * 1600), "partial sums fit the workspace");
        hipLaunchKernelGGL(k_train_block, dim3(parts), dim3(256), 0, st, params, params_bf16, features, n_rows, target,
                           (char*)workspace);
        L_TRY(hipGetLastError());
        hipLaunchKernelGGL(k_gradient_sum, dim3((unsigned)(kParams / kSumEntries + 1)), dim3(256), 0, st, (const char*)workspace,
                           parts, 1.0 / (3.0 * (double)n_rows), grad, loss);
        L_TRY(hipGetLastError());
        return FF_OK;
    }
    const long F = FF_LEARN_FEATURES, H = FF_LEARN_HIDDEN, O = FF_LEARN_OUT_PAD;
    const long n = n_rows;
    // forward into the first half of the workspace, gradients of the
    // activations into the second half
    const Act t = carve(workspace, n);
    const Act d = carve((char*)workspace + act_bytes(n), n);
    float* split = (float*)((char*)workspace + 2 * act_bytes(n));
    L_TRY(launch_gemm(n_rows, H, F, features, F, 1, params_bf16 + kW1, H, 1, params + kB1, 1, t.h1, H, t.h1b, H, st));
    L_TRY(launch_gemm(n_rows, H, H, t.h1b, H, 1, params_bf16 + kW2, H, 1, params + kB2, 1, t.h2, H, t.h2b, H, st));
    L_TRY(launch_gemm(n_rows, O, H, t.h2b, H, 1, params_bf16 + kW3, O, 1, params + kB3, 0, t.y, O, nullptr, 0, st));
    // dY (FP32 in d.y, BF16 in d.h2b's first n*O entries), per-row errors in d.h1
    uint16_t* dyb = d.h2b;
    float* row_loss = d.h1;
    hipLaunchKernelGGL(k_mse, dim3((n_rows + 255) / 256), dim3(256), 0, st, n_rows, t.y, target, d.y, dyb, row_loss);
    L_TRY(hipGetLastError());
    hipLaunchKernelGGL(k_colsum, dim3(1), dim3(256), 0, st, n_rows, 1, row_loss, 1.0 / (3.0 * n), loss);
    L_TRY(hipGetLastError());
    // layer 3: dW3 = H2^T dY, db3 = colsum dY, dH2 = dY W3^T (masked by H2 > 0)
    L_TRY(launch_gemm(H, O, n_rows, t.h2b, 1, H, dyb, O, 1, nullptr, 0, grad + kW3, O, nullptr, 0, st, split,
                      kSplitFloats));
    hipLaunchKernelGGL(k_colsum, dim3(O), dim3(256), 0, st, n_rows, (int)O, d.y, 1.0, grad + kB3);
    L_TRY(hipGetLastError());
    L_TRY(launch_gemm(n_rows, H, O, dyb, O, 1, params_bf16 + kW3, 1, O, nullptr, 0, d.h2, H, nullptr, 0, st));
    hipLaunchKernelGGL(k_relu_back, dim3((unsigned)((n * H + 255) / 256)), dim3(256), 0, st, n * H, t.h2, d.h2, d.h2b);
    L_TRY(hipGetLastError());
    // layer 2: dW2 = H1^T dH2, db2, dH1 = dH2 W2^T (masked by H1 > 0)
    L_TRY(launch_gemm(H, H, n_rows, t.h1b, 1, H, d.h2b, H, 1, nullptr, 0, grad + kW2, H, nullptr, 0, st, split,
                      kSplitFloats));
    hipLaunchKernelGGL(k_colsum, dim3(H), dim3(256), 0, st, n_rows, (int)H, d.h2, 1.0, grad + kB2);
    L_TRY(hipGetLastError());
    L_TRY(launch_gemm(n_rows, H, H, d.h2b, H, 1, params_bf16 + kW2, 1, H, nullptr, 0, d.h1, H, nullptr, 0, st));
    hipLaunchKernelGGL(k_relu_back, dim3((unsigned)((n * H + 255) / 256)), dim3(256), 0, st, n * H, t.h1, d.h1, d.h1b);
    L_TRY(hipGetLastError());
    // layer 1: dW1 = X^T dH1, db1
    L_TRY(launch_gemm(F, H, n_rows, features, 1, F, d.h1b, H, 1, nullptr, 0, grad + kW1, H, nullptr, 0, st, split,
                      kSplitFloats));
    hipLaunchKernelGGL(k_colsum, dim3(H), dim3(256), 0, st, n_rows, (int)H, d.h1, 1.0, grad + kB1);
    L_TRY(hipGetLastError());
    return FF_OK;
}

ff_status ff_learn_adam(float* params, uint16_t* params_bf16, const float* grad, float* m, float* v, int32_t step,
                        float lr, float beta1, float beta2, float eps, void* stream) {
    g_learn_err.clear();
    if (!params || !grad || !m || !v || step < 1 || !(lr > 0.0f)) return lfail(FF_ERR_ARG, "bad Adam arguments");
    const float c1 = 1.0f - std::pow(beta1, (float)step), c2 = 1.0f - std::pow(beta2, (float)step);
    hipLaunchKernelGGL(k_adam, dim3((unsigned)((kParams + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                       (int)kParams, params, params_bf16, grad, m, v, lr, beta1, beta2, eps, c1, c2);
    L_TRY(hipGetLastError());
    return FF_OK;
}

ff_status ff_learn_displace(const double* xyz, const float* disp, int32_t n_atoms, double scale, double* out,
                            void* stream) {
    g_learn_err.clear();
    if (!xyz || !disp || !out || n_atoms < 1 || !std::isfinite(scale)) return lfail(FF_ERR_ARG, "bad arguments");
    const long n3 = 3L * n_atoms;
    hipLaunchKernelGGL(k_displace, dim3((unsigned)((n3 + 255) / 256)), dim3(256), 0, (hipStream_t)stream, n3, xyz,
                       disp, scale, out);
    L_TRY(hipGetLastError());
    return FF_OK;
}

ff_status ff_learn_to_bf16(const float* x, int64_t n, uint16_t* out, void* stream) {
    g_learn_err.clear();
    if (!x || !out || n < 1) return lfail(FF_ERR_ARG, "bad conversion arguments");
    hipLaunchKernelGGL(k_to_bf16, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream, (long)n, x,
                       out);
    L_TRY(hipGetLastError());
    return FF_OK;
}

ff_status ff_learn_delta(const double* x_start, const double* x_min, int32_t n_atoms, float* out, void* stream) {
    g_learn_err.clear();
    if (!x_start || !x_min || !out || n_atoms < 1) return lfail(FF_ERR_ARG, "bad delta arguments");
    const long n3 = 3L * n_atoms;
    hipLaunchKernelGGL(k_delta, dim3((unsigned)((n3 + 255) / 256)), dim3(256), 0, (hipStream_t)stream, n3, x_start,
                       x_min, out);
    L_TRY(hipGetLastError());
    return FF_OK;
}

ff_status ff_learn_gather_rows(const void* src, const int32_t* idx, int32_t n_rows, int32_t row_bytes, void* dst,
                               void* stream) {
    g_learn_err.clear();
    if (!src || !idx || !dst || n_rows < 1 || row_bytes < 4 || (row_bytes & 3))
        return lfail(FF_ERR_ARG, "bad gather arguments");
    const int words = row_bytes / 4;
    const long tot = (long)n_rows * words;
    hipLaunchKernelGGL(k_gather, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                       (const uint32_t*)src, idx, (long)n_rows, words, (uint32_t*)dst);
    L_TRY(hipGetLastError());
    return FF_OK;
}

ff_status ff_learn_select(int32_t n_sys, int32_t n_total, const double* x_old, const double* x_new,
                          const double* e_old, const double* e_new, const int32_t* atom_sys, double* out,
                          int32_t* chosen, double* e_out, void* stream) {
    g_learn_err.clear();
    if (n_sys < 1 || n_total < 1 || !x_old || !x_new || !e_old || !e_new || !atom_sys || !out)
        return lfail(FF_ERR_ARG, "bad select arguments");
    hipStream_t st = (hipStream_t)stream;
    const long n3 = 3L * n_total;
    hipLaunchKernelGGL(k_select, dim3((unsigned)((n3 + 255) / 256)), dim3(256), 0, st, n3, x_old, x_new, e_old,
                       e_new, atom_sys, out);
    L_TRY(hipGetLastError());
    if (chosen || e_out) {
        hipLaunchKernelGGL(k_chosen, dim3((n_sys + 255) / 256), dim3(256), 0, st, n_sys, e_old, e_new, chosen,
                           e_out);
        L_TRY(hipGetLastError());
    }
    return FF_OK;
}

}  // extern "C"
