// Per-evaluation finalize (gradient gather, norms, energy total) and the
// optimizer's vector passes: trial point / direction construction and the
// accept pass (history vectors and their dot products).  In a pass that ends in
// a reduction each workgroup leaves partials, and a system's last workgroup sums
// them in a fixed order and runs the decision step (no workgroup waits for
// others).
#include "ff_decide.h"

namespace ff {

// Value of lane l ^ o of every 16 lanes' row (DPP), where the values already
// repeat with period 2 o: a rotation by o then reads the same as the exchange.
template <int O>
__device__ __forceinline__ double row_partner(double v) {
    constexpr int kCtrl = O == 1 ? 0xB1 /* quad_perm 1 0 3 2 */ : O == 2 ? 0x4E /* quad_perm 2 3 0 1 */
                                                                : 0x120 + O /* row_ror */;
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, kCtrl, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), kCtrl, 0xF, 0xF, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// op over a wavefront in the order of an xor butterfly (32, 16, ... 1), every
// lane receives it: register exchanges instead of twelve trips through the LDS
// crossbar, since the direction below is a chain of 21 such sums (with the
// decision on a copy in LDS, an accept pass of 512 atoms and ten pairs takes 16
// us instead of 22).
template <typename OP>
__device__ __forceinline__ double wave_reduce(double v, OP op) {
    auto halves = [&](auto swap) {
        const long long b = __double_as_longlong(v);
        const auto lo = swap((unsigned)b), hi = swap((unsigned)(b >> 32));
        v = op(__longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0])),
               __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1])));
    };
    halves([](unsigned x) { return __builtin_amdgcn_permlane32_swap(x, x, false, false); });
    halves([](unsigned x) { return __builtin_amdgcn_permlane16_swap(x, x, false, false); });
    v = op(v, row_partner<8>(v));
    v = op(v, row_partner<4>(v));
    v = op(v, row_partner<2>(v));
    return op(v, row_partner<1>(v));
}
__device__ __forceinline__ double wave_sum(double v) {
    return wave_reduce(v, [](double a, double b) { return a + b; });
}
__device__ __forceinline__ double wave_max(double v) {
    return wave_reduce(v, [](double a, double b) { return fmax(a, b); });
}

// Sum (or max for index 0 if first_is_max) of NV per-thread values over a
// 256-thread block; thread 0 receives the totals in out[].
template <int NV>
__device__ __forceinline__ void block_reduce(double (&v)[NV], bool first_is_max, double* out) {
    __shared__ double s[kFinBlock / 64][NV > 0 ? NV : 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const double r = (k == 0 && first_is_max) ? wave_max(v[k]) : wave_sum(v[k]);
        if (lane == 0) s[wave][k] = r;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            double r = s[0][k];
            for (int w = 1; w < kFinBlock / 64; ++w) r = (k == 0 && first_is_max) ? fmax(r, s[w][k]) : r + s[w][k];
            out[k] = r;
        }
    }
    __syncthreads();
}

// -------------------------------------------------------- L-BFGS direction
// Coefficients of the L-BFGS direction r = -H g (Algorithm 3) in the basis
// {s_0..s_{n-1}, y_0..y_{n-1}, g} of the stored pairs (oldest first) and the
// current gradient, from the Gram matrix of that basis: the two loops of the
// recursion act on coefficient vectors, every inner product becomes a row of
// the Gram matrix times the coefficients.  The workgroup copies the active
// (2n+1)^2 block into LDS; the first wavefront runs the loops, one wavefront
// sum per inner product (lane k holds coefficients k and k + 64).  On a
// descent direction (<g, r> < 0) the terms of r and |r| are written to the
// control block and lb_ready = 1, otherwise lb_ready = -1.  Every thread of
// the workgroup calls this; hist_n >= 1.
__device__ void lbfgs_direction_block(CtlState* c, const double* gram) {
    __shared__ double gs[kGramDim * kGramDim];
    __shared__ double cs[kGramDim];
    __shared__ int pos[kGramDim];
    const int n = c->hist_n;
    const int nb = 2 * n + 1;
    for (int k = threadIdx.x; k < nb; k += blockDim.x)
        pos[k] = k < n ? gpos_s(ring_slot(c, k)) : (k < 2 * n ? gpos_y(ring_slot(c, k - n)) : kGposG);
    __syncthreads();
    for (int e = threadIdx.x; e < nb * nb; e += blockDim.x) {
        const int r = e / nb, q = e - r * nb;
        gs[e] = gram[pos[r] * kGramDim + pos[q]];
    }
    __syncthreads();
    if (threadIdx.x >= 64) return;
    const int l = threadIdx.x, l2 = l + 64;
    double c0 = l == 2 * n ? -1.0 : 0.0;     // coefficient of basis element l
    double c1 = l2 == 2 * n ? -1.0 : 0.0;    // ... and of l + 64
    const double rho_l = l < n ? c->rho[ring_slot(c, l)] : 0.0;
    auto row_times_coef = [&](int r) {
        double v = 0.0;
        if (l < nb) v = gs[r * nb + l] * c0;
        if (l2 < nb) v += gs[r * nb + l2] * c1;
        return wave_sum(v);
    };
    double alpha_l = 0.0;
    for (int i = n - 1; i >= 0; --i) {             // newest to oldest
        const double a = __shfl(rho_l, i, 64) * row_times_coef(i);
        if (l == i) alpha_l = a;
        if (l == n + i) c0 -= a;
        if (l2 == n + i) c1 -= a;
    }
    const double gamma = gs[(n - 1) * nb + (2 * n - 1)] / gs[(2 * n - 1) * nb + (2 * n - 1)];
    c0 *= gamma;
    c1 *= gamma;
    for (int i = 0; i < n; ++i) {                  // oldest to newest
        const double b = __shfl(rho_l, i, 64) * row_times_coef(n + i);
        const double ai = __shfl(alpha_l, i, 64);
        if (l == i) c0 += ai - b;
    }
    const double gr = row_times_coef(2 * n);       // <g, r>
    if (l < nb) cs[l] = c0;
    if (l2 < nb) cs[l2] = c1;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // |r|^2 = c^T G c
    double part = 0.0;
    if (l < nb && c0 != 0.0) {
        double t = 0.0;
        for (int q = 0; q < nb; ++q) t += gs[l * nb + q] * cs[q];
        part = c0 * t;
    }
    if (l2 < nb && c1 != 0.0) {
        double t = 0.0;
        for (int q = 0; q < nb; ++q) t += gs[l2 * nb + q] * cs[q];
        part += c1 * t;
    }
    const double nrm2 = wave_sum(part);
    const bool ok = gr < 0.0 && nrm2 > 0.0 && isfinite(nrm2);
    if (ok) {
        auto term = [&](int k, double coef) {
            c->term_vec[k] = k < n ? c->hist_s[ring_slot(c, k)]
                           : (k < 2 * n ? c->hist_y[ring_slot(c, k - n)] : V_G0 + c->cur);
            c->term_coef[k] = coef;
        };
        if (l < nb) term(l, c0);
        if (l2 < nb) term(l2, c1);
    }
    if (l == 0) {
        if (ok) {
            c->n_terms = nb;
            c->dir_scale = sqrt(nrm2);
        }
        c->lb_ready = ok ? 1 : -1;
    }
}

// ------------------------------------------------------------------ finalize
// Partial rows in flight per wavefront of k_finalize, which is bound by their
// latency (10,000 atoms, FP32 rows: 10.5 us with eight, 12.1 with four; 16 are
// no faster, and slower in batches: 28 us against 22 for 96 chains of 4,000).
constexpr int kFlight = 8;
constexpr int kSlots = 3;        // bonded-term slots a thread fetches at a time

// Partials that a pass's workgroups leave for the last one of them: stored and
// read at device scope, past the caches of the XCDs.
__device__ __forceinline__ void put_partial(double* p, double v) {
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), (unsigned long long)__double_as_longlong(v),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double get_partial(const double* p) {
    return __longlong_as_double((long long)__hip_atomic_load(reinterpret_cast<const unsigned long long*>(p),
                                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// True in the last of a pass's n workgroups to get here (all threads; thread 0
// has put the workgroup's partials before).  It goes on with the reduction,
// instead of a launch of its own.  No workgroup counts before all of its
// wavefronts are here: the last one rewrites the control block that they read
// on their way.  The partials are in memory once their stores are acknowledged,
// so the counter needs no release, which would write back the XCD's whole L2
// from every workgroup.  FP64 evaluations with the launch, with the last
// workgroup, and with a release: 512 atoms 17.0, 16.0, 15.8 us; 96 chains of
// 200-4,000 atoms 205, 206, 248 us.
__device__ __forceinline__ bool last_workgroup(uint32_t* ticket, int n) {
    __shared__ int last;
    __syncthreads();
    if (threadIdx.x == 0) {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0x0f70);          // vmcnt(0)
        asm volatile("" ::: "memory");
        last = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)n - 1;
        if (last) *ticket = 0u;
    }
    __syncthreads();
    return last != 0;
}

// A control block's state between memory and LDS, by a whole workgroup: the
// decision step is a chain of small dependent accesses by one thread.
__device__ __forceinline__ void copy_state(CtlState* to, const CtlState* from) {
    for (int k = threadIdx.x; k < (int)(sizeof(CtlState) / sizeof(uint64_t)); k += kFinBlock)
        reinterpret_cast<uint64_t*>(to)[k] = reinterpret_cast<const uint64_t*>(from)[k];
}

// Pair partials of one 64-atom tile t of I-block `row`, summed over its
// partial rows in a fixed order.  The tile's rows are the i-side partials
// of every chunk of its I-block, then the j-side partials of every unit that
// holds tile t (I-blocks row0..row; in the FP64 table a unit whose tile is cut
// into parts has a row for each).  Each row is 192 contiguous values
// (64 atoms x xyz); wavefront w of the workgroup sums rows w, w+4, ... (lane
// l holds values l, l+64, l+128), the four wavefront sums are then added in
// order.  T is the storage type of the partials (FP32 mode: float).
template <typename T>
__device__ __forceinline__ void gather_tile(const Args& a, const SysInfo& si, int row, int t,
                                            double* tot /* LDS [192] */, double (*part)[3 * kTile] /* LDS */) {
    constexpr int kWaves = kFinBlock / 64;
    const Layout& L = a.L;
    const RowInfo* R = at<RowInfo>(a.ws, L.off_rows);
    const T* Pi = at<T>(a.ws, L.off_pi);
    const T* Pj = at<T>(a.ws, L.off_pj);
    const int row0 = si.row0;
    const RowInfo ri = R[row];
    const int il0 = t * kTile - row * L.block;
    constexpr int tab = sizeof(T) == 4 ? 0 : 1;          // chunk table of the kernel that wrote Pi
    const int per = tab == 0 ? 1 : unit_rows(L.split);   // rows of a unit
    const int n_i = ri.n_chunks[tab], nseg = n_i + (row - row0 + 1) * per;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // Units of a system are numbered row by row, local row r holding tiles
    // r*B/64 .. nt-1, so the unit of (row r, tile tl) has a closed form and
    // the addresses need no table loads.
    const long long u0 = R[row0].unit_start;
    const long long nt = si.np / kTile, b64 = L.block / kTile;
    const long long tl = t - si.aoff / kTile;
    auto seg = [&](int sg) -> const T* {
        if (sg < n_i) return Pi + ((size_t)(ri.chunk_start[tab] + sg) * L.block + il0) * 3;
        const int q = sg - n_i;
        const long long r = per == 1 ? q : q / per;
        const long long unit = u0 + r * nt - b64 * r * (r - 1) / 2 + (tl - r * b64);
        return Pj + (size_t)(per == 1 ? unit : unit * per + (q - r * per)) * (3 * kTile);
    };
    double acc[3] = {};
    // kFlight rows in flight per wavefront, added in row order; past the last
    // row nothing is added (0.0 to a sum that began at 0.0)
    for (int sg = wave; sg < nseg; sg += kFlight * kWaves) {
        T v[kFlight][3];
#pragma unroll
        for (int f = 0; f < kFlight; ++f) {
            const T* p = seg(min(sg + f * kWaves, nseg - 1)) + lane;
#pragma unroll
            for (int k = 0; k < 3; ++k) v[f][k] = p[64 * k];
        }
#pragma unroll
        for (int f = 0; f < kFlight; ++f)
#pragma unroll
            for (int k = 0; k < 3; ++k) acc[k] += sg + f * kWaves < nseg ? (double)v[f][k] : 0.0;
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) part[wave][lane + 64 * k] = acc[k];
    __syncthreads();
    if (threadIdx.x < 3 * kTile) {
        double v = part[0][threadIdx.x];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) v += part[w][threadIdx.x];
        tot[threadIdx.x] = v;
    }
    __syncthreads();
}

// floor(count * b / nb) for b <= nb (a 64-bit division costs 150 instructions).
__device__ __forceinline__ int share_begin(int count, int b, int nb) {
    const unsigned q = (unsigned)count / (unsigned)nb, r = (unsigned)count % (unsigned)nb;
    const unsigned rest = nb < 65536 ? r * (unsigned)b / (unsigned)nb : (unsigned)((unsigned long long)r * b / nb);
    return (int)(q * (unsigned)b + rest);
}

// Share of tile `blk` in the energies of a system's pair chunks (table `tab`)
// and bonded blocks, per thread.
__device__ __forceinline__ double energy_share(const Args& a, const SysInfo& si, int blk, int tab) {
    const double* ep = at<double>(a.ws, a.L.off_ep) + si.chunk0[tab];
    const double* eb = at<double>(a.ws, a.L.off_eb) + si.eb0;
    const int nb = si.fin_blocks, nc = si.n_chunks[tab];
    const int p0 = share_begin(nc, blk, nb), p1 = share_begin(nc, blk + 1, nb);
    const int q0 = share_begin(si.bonded_blocks, blk, nb), q1 = share_begin(si.bonded_blocks, blk + 1, nb);
    double e = 0.0;
    for (int k = p0 + (int)threadIdx.x; k < p1; k += kFinBlock) e += ep[k];
    for (int k = q0 + (int)threadIdx.x; k < q1; k += kFinBlock) e += eb[k];
    return e;
}

// The decision of k_finalize's last workgroup is a call: inlined, it costs the
// gather of every tile registers and 96 chains of 200-4,000 atoms 1 % of an
// evaluation.
__device__ __attribute__((noinline)) void decide(CtlState* c) { after_eval(c); }

// One workgroup per 64-atom tile of a system: gradient = pair partials of
// the tile (gather_tile) + the bonded-term slots of each atom (staged through
// LDS, added in slot order).  Per-workgroup partials: max |g|, |g|^2,
// optionally <g_base, d>, and a share of the pair-workgroup and bonded-block
// energies, which the system's last workgroup adds up.  Grid: every tile of
// every system (flat, map_fin).
__global__ void __launch_bounds__(kFinBlock) k_finalize(Args a) {
    const Layout& L = a.L;
    const int2 mb = at<int2>(a.ws, L.off_map_fin)[blockIdx.x];
    const int sys = mb.x, blk = mb.y;                    // system and its tile
    const SysInfo si = sys_info(a)[sys];
    Ctl* c = ctl_at(a, sys);
    if (!a.direct && (c->action != ACT_EVAL || c->target < 0 || c->target >= kNumSlots)) return;
    double* G = a.direct ? (a.g_out ? a.g_out + 3 * (size_t)si.uoff : nullptr) : vec(a, V_G0 + c->target, si);
    const bool want_slope = !a.direct && c->want_slope;
    const int t = si.aoff / kTile + blk;                 // global tile
    const int row = t * kTile / L.block;                 // its I-block
    __shared__ double tot[3 * kTile];
    __shared__ double part[kFinBlock / 64][3 * kTile];
    __shared__ double fbv[kSlots * kFinBlock][3];
    const bool p32 = a.direct ? a.direct_prec == 1 : c->prec == 1;
    // bonded-term slots of the tile's atoms: contiguous in the incidence list
    const int* inc0 = at<int>(a.ws, L.off_inc_start);
    const int* inc = at<int>(a.ws, L.off_inc);
    const double* FB = at<double>(a.ws, L.off_fb);
    const int ga = t * kTile + (int)threadIdx.x;         // global padded atom (threads < 64)
    const int k_lo = inc0[t * kTile], k_hi = inc0[t * kTile + kTile];
    int my_lo = 0, my_hi = 0;
    if (threadIdx.x < kTile) {
        my_lo = inc0[ga];
        my_hi = inc0[ga + 1];
    }
    // kSlots slots of a thread from `base` (past the last slot its values again,
    // which nothing reads); the first ones are on their way while the partial
    // rows are summed
    double fb[kSlots][3];
    auto fetch = [&](int base) {
#pragma unroll
        for (int m = 0; m < kSlots; ++m) {
            const double* p = FB + 3 * (size_t)inc[min(base + m * kFinBlock + (int)threadIdx.x, k_hi - 1)];
            fb[m][0] = p[0]; fb[m][1] = p[1]; fb[m][2] = p[2];
        }
    };
    if (k_lo < k_hi) fetch(k_lo);
    double e = energy_share(a, si, blk, p32 ? 0 : 1);
    if (p32) gather_tile<float>(a, si, row, t, tot, part);
    else gather_tile<double>(a, si, row, t, tot, part);
    double gx = 0.0, gy = 0.0, gz = 0.0;
    if (threadIdx.x < kTile) {
        gx = tot[3 * threadIdx.x];
        gy = tot[3 * threadIdx.x + 1];
        gz = tot[3 * threadIdx.x + 2];
    }
    for (int base = k_lo; base < k_hi; base += kSlots * kFinBlock) {
        if (base > k_lo) fetch(base);
#pragma unroll
        for (int m = 0; m < kSlots; ++m)
#pragma unroll
            for (int q = 0; q < 3; ++q) fbv[m * kFinBlock + (int)threadIdx.x][q] = fb[m][q];
        __syncthreads();
        if (threadIdx.x < kTile) {
            const int end = min(my_hi, base + kSlots * kFinBlock);
            for (int q = max(my_lo, base); q < end; ++q) {
                gx += fbv[q - base][0]; gy += fbv[q - base][1]; gz += fbv[q - base][2];
            }
        }
        __syncthreads();
    }
    const int atom = blk * kTile + (int)threadIdx.x;          // local atom
    const bool real = threadIdx.x < kTile && atom < si.n;
    if (!real) gx = gy = gz = 0.0;
    if (real && G) { G[3 * (size_t)atom] = gx; G[3 * (size_t)atom + 1] = gy; G[3 * (size_t)atom + 2] = gz; }
    double v[4];
    v[0] = fmax(fabs(gx), fmax(fabs(gy), fabs(gz)));
    if (isnan(gx) || isnan(gy) || isnan(gz)) v[0] = __builtin_inf();
    v[1] = fma(gz, gz, fma(gy, gy, gx * gx));
    v[2] = 0.0;
    if (want_slope && real) {
        const double* gb = vec(a, V_G0 + c->slope_slot, si);
        const double* d = vec(a, V_D, si);
        const size_t o = 3 * (size_t)atom;
        v[2] = fma(gb[o + 2], d[o + 2], fma(gb[o], d[o], gb[o + 1] * d[o + 1]));
    }
    v[3] = e;
    double* red = at<double>(a.ws, L.off_red) + si.red0;
    double tr[4];
    block_reduce<4>(v, true, tr);
    if (threadIdx.x == 0)
        for (int k = 0; k < 4; ++k) put_partial(red + 4 * blk + k, tr[k]);

    // Last workgroup of the system: totals in a fixed order, then E, the norms
    // and the decision step (ff_energy_grad: the energy only).
    if (!last_workgroup(&c->fin_ticket, si.fin_blocks)) return;
    double w[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int b = threadIdx.x; b < si.fin_blocks; b += kFinBlock) {
        w[0] = fmax(w[0], get_partial(red + 4 * b));
        w[1] += get_partial(red + 4 * b + 1);
        w[2] += get_partial(red + 4 * b + 2);
        w[3] += get_partial(red + 4 * b + 3);
    }
    static_assert(sizeof(CtlState) <= sizeof fbv, "the state takes the place of the slots");
    CtlState& state = *reinterpret_cast<CtlState*>(fbv);
    if (!a.direct) copy_state(&state, c);
    double gt[4];
    block_reduce<4>(w, true, gt);
    if (a.direct) {
        if (threadIdx.x == 0) {
            if (a.e_out) a.e_out[sys] = gt[3];
            if (a.g2_out) a.g2_out[sys] = gt[1];
        }
        return;
    }
    if (threadIdx.x == 0) {
        const int tg = state.target;
        state.e[tg] = gt[3];
        state.ginf[tg] = gt[0];
        state.g2[tg] = gt[1];
        if (want_slope) state.slope = gt[2];
        decide(&state);
    }
    __syncthreads();
    copy_state(c, &state);
}

// ------------------------------------------------------------------- prepare
// Builds the point to evaluate: a trial x + h d, the direction itself
// (d = r / |r| with r a linear combination of stored vectors) followed by the
// trial, or the FGM momentum point.  Rounding is kept explicit (no
// contraction) so that trial points are reproducible.
__global__ void __launch_bounds__(kFinBlock) k_prepare(Args a) {
    const int2 mb = at<int2>(a.ws, a.L.off_map_vec)[blockIdx.x];
    const int sys = mb.x;
    const SysInfo si = sys_info(a)[sys];
    const Ctl* c = ctl_at(a, sys);
    if (c->action != ACT_EVAL || c->point_mode == PM_USE) return;
    if (c->target < 0 || c->target >= kNumSlots || c->base < 0 || c->base >= kNumSlots) return;
    const int pm = c->point_mode;
    if ((pm == PM_MOMENTUM || pm == PM_HB || pm == PM_OGM_Y) && (c->prev < 0 || c->prev >= kNumSlots)) return;
    const int n3 = 3 * si.n;
    const int i = mb.y * kFinBlock + threadIdx.x;
    if (i >= n3) return;
    double* xt = vec(a, V_X0 + c->target, si);
    const double* xb = vec(a, V_X0 + c->base, si);
    if (pm == PM_MOMENTUM) {
        const double* xp = vec(a, V_X0 + c->prev, si);
        xt[i] = __dadd_rn(xb[i], __dmul_rn(c->beta, __dsub_rn(xb[i], xp[i])));
        return;
    }
    if (pm == PM_HB) {
        const double* xp = vec(a, V_X0 + c->prev, si);
        const double* gb = vec(a, V_G0 + c->base, si);
        xt[i] = __dadd_rn(__dsub_rn(xb[i], __dmul_rn(c->h, gb[i])), __dmul_rn(c->beta, __dsub_rn(xb[i], xp[i])));
        return;
    }
    double* d = vec(a, V_D, si);
    double di;
    if (pm == PM_DIR_TRIAL || pm == PM_OGM_Y) {
        double r = __dmul_rn(c->term_coef[0], vec(a, c->term_vec[0], si)[i]);
#pragma unroll 4
        for (int k = 1; k < c->n_terms; ++k) r = __dadd_rn(r, __dmul_rn(c->term_coef[k], vec(a, c->term_vec[k], si)[i]));
        if (c->write_r) vec(a, V_R, si)[i] = r;
        di = __ddiv_rn(r, c->dir_scale);
        d[i] = di;
    } else {
        di = d[i];
    }
    if (pm == PM_OGM_Y) {
        const double* xa = vec(a, V_X0 + c->prev, si);
        xt[i] = __dadd_rn(__dmul_rn(1.0 - c->beta, xb[i]), __dmul_rn(c->beta, xa[i]));
        return;
    }
    xt[i] = __dadd_rn(xb[i], __dmul_rn(c->h, di));
}

// -------------------------------------------------------------------- accept
// After a successful line search: method-specific vectors and dot products.
//  CG:     <g_new, g_old>, <g_new, r_old>, <r_old, g_old>
//  L-BFGS: s = x_new - x_old and y = g_new - g_old (written to the spare
//          history vectors), <s,y> <y,y> <s,s> <g,s> <g,y> <g,g> and, for
//          the pair in every occupied history slot q, <s,S_q> <s,Y_q>
//          <y,S_q> <y,Y_q> <g,S_q> <g,Y_q>.
// Grid: (accept workgroups of every system (flat, map_acc), 1 + largest
// L-BFGS memory).  Row 0 computes the first group of six, row r >= 1 the six
// products with the pair in slot r-1 (s and y are recomputed from the point
// vectors in every row, with the same arithmetic); each workgroup strides over
// its share of the 3N elements and writes one partial per product
// (the system's last workgroup adds them up in workgroup order, then makes the
// method update and the next iteration; L-BFGS: the coefficients of the next
// direction are computed by the workgroup first).
__global__ void __launch_bounds__(kFinBlock) k_accept(Args a) {
    const int2 mb = at<int2>(a.ws, a.L.off_map_acc)[blockIdx.x];
    const int sys = mb.x, bx = mb.y;
    const SysInfo si = sys_info(a)[sys];
    Ctl* c = ctl_at(a, sys);
    if (!c->accept) return;
    const int n3 = 3 * si.n;
    const int method = c->p.method;
    const int row = blockIdx.y;
    // the control block is fixed until the pass's last workgroup is here
    const int rows = c->acc_rows;
    const bool active = row < rows;
    double* red = at<double>(a.ws, a.L.off_red) + si.red0;
    const int nbx = si.acc_bx;
    if (active) {
        double v[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        const double* xn = vec(a, V_X0 + c->acc_new, si);
        const double* xo = vec(a, V_X0 + c->acc_old, si);
        const double* gn = vec(a, V_G0 + c->acc_new, si);
        const double* go = vec(a, V_G0 + c->acc_old, si);
        const int stride = nbx * kFinBlock;
        if (method == M_OGM) {
            // S += t_{k+1} g_new (S is the anchor's gradient after a restart)
            const double* src = c->ogm_s_anchor ? vec(a, V_G0 + c->prev_x, si) : vec(a, V_R, si);
            double* S = vec(a, V_R, si);
            const double t = c->ogm_t_next;
#pragma unroll 4
            for (int i = bx * kFinBlock + threadIdx.x; i < n3; i += stride) {
                const double sn = __dadd_rn(src[i], __dmul_rn(t, gn[i]));
                S[i] = sn;
                v[0] += gn[i] * sn;
                v[1] += sn * sn;
            }
        } else if (method == M_CG) {
            const double* r = vec(a, V_R, si);
#pragma unroll 4
            for (int i = bx * kFinBlock + threadIdx.x; i < n3; i += stride) {
                v[0] += gn[i] * go[i];
                v[1] += gn[i] * r[i];
                v[2] += r[i] * go[i];
            }
        } else if (row == 0) {
            double* ss = vec(a, c->spare_s, si);
            double* yy = vec(a, c->spare_y, si);
#pragma unroll 4
            for (int i = bx * kFinBlock + threadIdx.x; i < n3; i += stride) {
                const double s = __dsub_rn(xn[i], xo[i]);
                const double g = gn[i];
                const double y = __dsub_rn(g, go[i]);
                ss[i] = s;
                yy[i] = y;
                v[0] += s * y; v[1] += y * y; v[2] += s * s;
                v[3] += g * s; v[4] += g * y; v[5] += g * g;
            }
        } else {
            const double* S = vec(a, c->hist_s[row - 1], si);
            const double* Y = vec(a, c->hist_y[row - 1], si);
#pragma unroll 4
            for (int i = bx * kFinBlock + threadIdx.x; i < n3; i += stride) {
                const double s = __dsub_rn(xn[i], xo[i]);
                const double g = gn[i];
                const double y = __dsub_rn(g, go[i]);
                const double Si = S[i], Yi = Y[i];
                v[0] += s * Si; v[1] += s * Yi; v[2] += y * Si;
                v[3] += y * Yi; v[4] += g * Si; v[5] += g * Yi;
            }
        }
        double tot[6];
        block_reduce<6>(v, false, tot);
        if (threadIdx.x == 0)
            for (int k = 0; k < 6; ++k) put_partial(red + ((size_t)row * nbx + bx) * 6 + k, tot[k]);
    }
    if (!last_workgroup(&c->acc_ticket, nbx * (int)gridDim.y)) return;
    __shared__ double dots[kMaxDots];
    const int nd = method == M_LBFGS || method == M_OGM ? 6 * rows : (method == M_CG ? 3 : 0);
    for (int k = threadIdx.x; k < nd; k += kFinBlock) {
        const int r = k / 6, q = k - 6 * r;
        double acc = 0.0;
#pragma unroll 16
        for (int b = 0; b < nbx; ++b) acc += get_partial(red + ((size_t)r * nbx + b) * 6 + q);
        dots[k] = acc;
    }
    __shared__ CtlState state;
    copy_state(&state, c);
    __syncthreads();
    if (method == M_LBFGS) {
        if (lbfgs_update(&state, c->gram, dots)) lbfgs_direction_block(&state, c->gram);
    } else if (threadIdx.x == 0) {
        accept_update(&state, dots);
    }
    __syncthreads();
    if (threadIdx.x == 0) accept_finish(&state);
    __syncthreads();
    copy_state(c, &state);
}

// ---------------------------------------------------------------------- kick
// Starts (or resumes) a minimization: one thread sets up the control block.
// One workgroup per system (system 0 keeps the per-iteration trace).
__global__ void k_kick(Args a, MinParamsDev p, int resume, double* trace, int trace_cap) {
    const int sys = blockIdx.x;
    Ctl* c = ctl_at(a, sys);
    if (threadIdx.x == 0) c->fin_ticket = c->acc_ticket = 0u;
    if (resume) {
        // continue where the previous call stopped; the L-BFGS direction is
        // recomputed from the stored pairs exactly as after an accept
        __shared__ int need_dir;
        if (threadIdx.x == 0) {
            c->batch = at<BatchState>(a.ws, a.L.off_batch);
            c->n_atoms = sys_info(a)[sys].n;
            const bool same_memory = c->p.method == M_LBFGS && p.method == M_LBFGS && c->hist_m == p.m;
            c->p = p;
            if (!same_memory) lbfgs_clear(c);
            c->done = 0;
            c->iters_limit = c->iters + p.max_iter;
            c->trace_ptr = sys == 0 ? trace : nullptr;
            c->trace_cap = trace_cap;
            c->n_trace = 0;
            c->iters_base = c->iters;
            c->fp32_released = 0;
            if (c->escalated) release_fp32(c);
            need_dir = p.method == M_LBFGS && c->hist_n > 0;
        }
        __syncthreads();
        if (need_dir) lbfgs_direction_block(c, c->gram);
        __syncthreads();
        if (threadIdx.x == 0) begin_iteration(c);
        return;
    }
    if (threadIdx.x != 0) return;
    if (sys != 0) trace = nullptr;
    c->batch = at<BatchState>(a.ws, a.L.off_batch);
    c->n_atoms = sys_info(a)[sys].n;
    c->p = p;
    c->phase = PH_START;
    c->done = 0;
    c->term = -1;
    c->iters = 0;
    c->iters_base = 0;
    c->evals = 0;
    c->evals64 = 0;
    c->iters_limit = p.max_iter;
    c->cur = 0;
    c->prev_x = (p.method == M_FGM || p.method == M_HB || p.method == M_OGM) ? 0 : -1;
    c->ogm_t = 1.0;
    c->ogm_s_anchor = 1;
    c->best = -1;
    c->w = -1;
    c->ls_base = -1;
    c->ls_best = -1;
    c->prec_now = p.precision;
    c->escalated = 0;
    c->stall32 = 0;
    c->fp32_released = 0;
    c->h_prev = p.h_init;
    c->steepest = 1;
    c->theta_prev = 1.0;
    c->fgm_beta = 0.0;
    c->cg_beta = 0.0;
    c->accept = 0;
    c->result_slot = 0;
    lbfgs_clear(c);
    for (int s = 0; s < kNumSlots; ++s) c->slot_prec[s] = -1;
    c->trace_ptr = trace;
    c->trace_cap = trace_cap;
    c->n_trace = 0;
    request_eval(c, PM_USE, 0, 0);
}

__device__ __forceinline__ void reset_batch(BatchState* b) {
    b->n_done = 0u;
    b->evals = 0u;
    b->n_fp64 = 0u;
}

// Zeroes the batch counters (before a minimization starts).
__global__ void k_reset_batch(Args a) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    reset_batch(at<BatchState>(a.ws, a.L.off_batch));
}

// Caller's coordinates into slot 0 (before a minimization starts) and the
// result slot's back.  Grid: flat over every system's 3n elements (map_vec).
__global__ void __launch_bounds__(kFinBlock) k_load_points(Args a, const double* xyz) {
    const int2 mb = at<int2>(a.ws, a.L.off_map_vec)[blockIdx.x];
    const SysInfo si = sys_info(a)[mb.x];
    const int i = mb.y * kFinBlock + threadIdx.x;
    if (i < 3 * si.n) vec(a, V_X0, si)[i] = xyz[3 * (size_t)si.uoff + i];
}

__global__ void __launch_bounds__(kFinBlock) k_store_results(Args a, double* xyz, ResultDev* res) {
    const int2 mb = at<int2>(a.ws, a.L.off_map_vec)[blockIdx.x];
    const SysInfo si = sys_info(a)[mb.x];
    const Ctl* c = ctl_at(a, mb.x);
    const int slot = c->result_slot;
    const int i = mb.y * kFinBlock + threadIdx.x;
    if (i < 3 * si.n) xyz[3 * (size_t)si.uoff + i] = vec(a, V_X0 + slot, si)[i];
    if (i == 0)
        res[mb.x] = ResultDev{c->term, c->iters - c->iters_base, c->evals, c->evals64, c->e[slot], c->ginf[slot],
                              c->g2[slot]};
}

// The batch counters to pinned host memory.
__global__ void k_report(Args a, BatchState* to) {
    if (threadIdx.x == 0) *to = *at<BatchState>(a.ws, a.L.off_batch);
}

// Marks every system idle and zeroes the batch counters (after ff_create).
__global__ void k_reset_ctl(Args a) {
    if (threadIdx.x != 0) return;
    if (blockIdx.x == 0) reset_batch(at<BatchState>(a.ws, a.L.off_batch));
    Ctl* c = ctl_at(a, blockIdx.x);
    c->batch = nullptr;
    c->action = ACT_NONE;
    c->accept = 0;
    c->done = 1;
    c->phase = PH_IDLE;
    c->iters = 0;
    c->fin_ticket = 0;
    c->acc_ticket = 0;
}

// Point of the energy profile: x + t u with u = -g / |g| per system (u = 0
// where g = 0), all in the caller's concatenated layout.  Grid: flat over
// every system's 3n elements (map_vec).
__global__ void __launch_bounds__(kFinBlock) k_profile_point(Args a, const double* x, const double* g,
                                                             const double* g2, double t, double* xt) {
    const int2 mb = at<int2>(a.ws, a.L.off_map_vec)[blockIdx.x];
    const SysInfo si = sys_info(a)[mb.x];
    const int i = mb.y * kFinBlock + threadIdx.x;
    if (i >= 3 * si.n) return;
    const size_t o = 3 * (size_t)si.uoff + i;
    const double nrm = sqrt(g2[mb.x]);
    const double u = nrm > 0.0 ? __ddiv_rn(-g[o], nrm) : 0.0;
    xt[o] = __dadd_rn(x[o], __dmul_rn(t, u));
}

hipError_t launch_profile_point(const Args& a, const double* x, const double* g, const double* g2, double t,
                                double* xt, hipStream_t s) {
    hipLaunchKernelGGL(k_profile_point, dim3(a.L.n_vec_blocks), dim3(kFinBlock), 0, s, a, x, g, g2, t, xt);
    return hipGetLastError();
}

hipError_t launch_finalize(const Args& a, hipStream_t s) {
    hipLaunchKernelGGL(k_finalize, dim3(a.L.n_fin_blocks), dim3(kFinBlock), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_cycle_vec(const Args& a, int which, hipStream_t s) {
    if (which == 0)
        hipLaunchKernelGGL(k_prepare, dim3(a.L.n_vec_blocks), dim3(kFinBlock), 0, s, a);
    else
        hipLaunchKernelGGL(k_accept, dim3(a.L.n_acc_blocks, a.L.acc_rows), dim3(kFinBlock), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_load_points(const Args& a, const double* xyz, hipStream_t s) {
    hipLaunchKernelGGL(k_load_points, dim3(a.L.n_vec_blocks), dim3(kFinBlock), 0, s, a, xyz);
    return hipGetLastError();
}

hipError_t launch_store_results(const Args& a, double* xyz, ResultDev* res, hipStream_t s) {
    hipLaunchKernelGGL(k_store_results, dim3(a.L.n_vec_blocks), dim3(kFinBlock), 0, s, a, xyz, res);
    return hipGetLastError();
}

hipError_t launch_report(const Args& a, BatchState* to, hipStream_t s) {
    hipLaunchKernelGGL(k_report, dim3(1), dim3(64), 0, s, a, to);
    return hipGetLastError();
}

hipError_t launch_kick(const Args& a, const MinParamsDev& p, int resume, double* trace, int trace_cap,
                       hipStream_t s) {
    hipLaunchKernelGGL(k_reset_batch, dim3(1), dim3(64), 0, s, a);
    hipLaunchKernelGGL(k_kick, dim3(a.L.n_sys), dim3(64), 0, s, a, p, resume, trace, trace_cap);
    return hipGetLastError();
}

hipError_t launch_reset(const Args& a, hipStream_t s) {
    hipLaunchKernelGGL(k_reset_ctl, dim3(a.L.n_sys), dim3(64), 0, s, a);
    return hipGetLastError();
}

}  // namespace ff
