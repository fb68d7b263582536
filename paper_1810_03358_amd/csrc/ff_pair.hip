// Nonbonded all-pairs energy and gradient (Coulomb + 12-6 Lennard-Jones with
// geometric mixing, section 2 of the paper) and the bonded terms (stretch,
// bend, OPLS torsion, section 2), for one evaluation point.
//
// Work decomposition.  Atoms are padded to np (multiple of 512) with
// zero-parameter atoms placed far away.  The upper triangle of the pair
// matrix is cut into units (I-block of B atoms) x (j-tile of 64 atoms), j-tile
// index t >= B*row/64; a chunk (a workgroup, or one of a workgroup's wavefronts)
// walks a run of j-tiles of one I-block, or in small FP64 systems a part of a
// tile.  Each lane keeps IPL i-atoms in registers; the j-tile sits in LDS
// twice in a row so that at step s lane l reads entry l+s (atom (l+s) mod 64)
// with an immediate offset.  The gradient on j is accumulated in a register
// that moves one lane down after every step (DPP wave rotation), so after 64
// steps every lane again holds the sum for "its" j.  Per-tile FP32 sums are
// folded into FP64; per-unit j sums and per-chunk i sums are written to
// partial buffers that the finalize kernel adds up in a fixed order, so the
// result is deterministic.  Newton's third law is used: every pair is
// computed once.
//
// Per pair, with per-atom factors prepared once per system
//   c12 = 2 sqrt(eps) sigma^6,  c6 = 2 sqrt(eps) sigma^3,  q^ = sqrt(C) q
// (so c12_i c12_j = 4 eps_ij sigma_ij^12, c6_i c6_j = 4 eps_ij sigma_ij^6,
//  q^_i q^_j = C q_i q_j), the terms of section 2 are
//   e12 = c12_i c12_j / r^12, e6 = c6_i c6_j / r^6, ec = q^_i q^_j / r
//   E  += e12 - e6 + ec
//   f   = (12 e12 - 6 e6 + ec) / r^2,  d = x_j - x_i
//   grad_i += f d,  grad_j -= f d.
// They are evaluated as follows, with the i-atom's factors held as 12 c12_i
// and 6 c6_i (s = 1/r^6, A = 12 c12_i c12_j, B = 6 c6_i c6_j):
//   u = A s - B                  (12 e12 - 6 e6 = u s)
//   f = (u s + ec) / r^2
//   L += (u - B) s               (12 e12 - 12 e6 = (u - B) s),  Ec += ec
// and E = L / 12 + Ec: 13 operations after 1/r instead of 16 for the direct
// form.  The Lennard-Jones and Coulomb sums are kept apart: one FP32 sum of
// both (or of 12 E) loses about 1e-6 of |E| at relaxed 10^4-atom chains.
#include "ff_internal.h"

namespace ff {

// Unroll of the 64-step j loop of the FP32 kernel: with one i-atom per lane
// four steps keep enough independent work in flight; with two the register
// budget of an unroll by four would cost a wavefront per SIMD (measured on
// the 50k chain: 1.05 ms with unroll 2 against 1.19 ms with 4 for 2 atoms per
// lane; 1.05 against 1.07 ms the other way round for 1 atom per lane).
template <int IPL>
constexpr int kUnroll32 = IPL == 1 ? 4 : 2;

#ifndef FF_DPP_ROTATE
#define FF_DPP_ROTATE 0x134   // wave_rol:1 -- lane l receives lane (l+1) mod 64
#endif

__device__ __forceinline__ float rotate_down(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), FF_DPP_ROTATE, 0xF, 0xF, false));
}
__device__ __forceinline__ double rotate_down(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)(b & 0xffffffffLL), FF_DPP_ROTATE, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), FF_DPP_ROTATE, 0xF, 0xF, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

__device__ __forceinline__ void load_pos(const double* X, int32_t atom, int32_t n, double* p) {
    if (atom < n) {
        p[0] = X[3 * (size_t)atom];
        p[1] = X[3 * (size_t)atom + 1];
        p[2] = X[3 * (size_t)atom + 2];
    } else {
        pad_position(atom, n, p);
    }
}

// ------------------------------------------------------------------ bonded
// Energy of bonded term t (bonds, then angles, then dihedrals; FP64) and its
// gradient on each of its atoms, written to the term's own slots (no scatter).
__device__ double bonded_term(const Args& a, const double* X, const SysInfo& si, int t) {
    const Layout& L = a.L;
    double e = 0.0;
    double* FB = at<double>(a.ws, L.off_fb);
    if (t < si.n_bonds) {
        t += si.bond0;
        const int2 b = at<int2>(a.ws, L.off_bond)[t];
        const double2 kp = at<double2>(a.ws, L.off_bondp)[t];   // (K, r0)
        double d[3], r2 = 0.0;
        for (int c = 0; c < 3; ++c) { d[c] = X[3 * b.x + c] - X[3 * b.y + c]; r2 += d[c] * d[c]; }
        const double r = sqrt(r2);
        const double dr = r - kp.y;
        e = kp.x * dr * dr;
        const double s = 2.0 * kp.x * dr / r;
        double* o = FB + 6 * (size_t)t;
        for (int c = 0; c < 3; ++c) { o[c] = s * d[c]; o[3 + c] = -s * d[c]; }
    } else if (t < si.n_bonds + si.n_angles) {
        const int k = t - si.n_bonds + si.angle0;
        const int* ia = at<int>(a.ws, L.off_angle) + 3 * k;
        const double2 kp = at<double2>(a.ws, L.off_anglep)[k];  // (K, theta0)
        double u[3], v[3];
        for (int c = 0; c < 3; ++c) {
            u[c] = X[3 * ia[0] + c] - X[3 * ia[1] + c];
            v[c] = X[3 * ia[2] + c] - X[3 * ia[1] + c];
        }
        // w = u x v; theta = atan2(|w|, u.v);
        // d theta/d x_i = (u x w)/(|u|^2 |w|), d theta/d x_k = -(v x w)/(|v|^2 |w|)
        const double w[3] = {u[1] * v[2] - u[2] * v[1], u[2] * v[0] - u[0] * v[2], u[0] * v[1] - u[1] * v[0]};
        const double nw = sqrt(w[0] * w[0] + w[1] * w[1] + w[2] * w[2]);
        const double uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
        const double vv = v[0] * v[0] + v[1] * v[1] + v[2] * v[2];
        const double uv = u[0] * v[0] + u[1] * v[1] + u[2] * v[2];
        const double th = atan2(nw, uv);
        const double dth = th - kp.y;
        e = kp.x * dth * dth;
        const double de = 2.0 * kp.x * dth;
        const double uxw[3] = {u[1] * w[2] - u[2] * w[1], u[2] * w[0] - u[0] * w[2], u[0] * w[1] - u[1] * w[0]};
        const double vxw[3] = {v[1] * w[2] - v[2] * w[1], v[2] * w[0] - v[0] * w[2], v[0] * w[1] - v[1] * w[0]};
        const double si = de / (uu * nw), sk = -de / (vv * nw);
        double* o = FB + 6 * (size_t)L.n_bonds + 9 * (size_t)k;
        for (int c = 0; c < 3; ++c) {
            const double gi = si * uxw[c], gk = sk * vxw[c];
            o[c] = gi;
            o[3 + c] = -(gi + gk);
            o[6 + c] = gk;
        }
    } else if (t < si.n_bonds + si.n_angles + si.n_dihedrals) {
        const int k = t - si.n_bonds - si.n_angles + si.dih0;
        const int* id = at<int>(a.ws, L.off_dih) + 4 * k;
        const double* V = at<double>(a.ws, L.off_dihp) + 4 * k;
        // F = x_a - x_b, G = x_b - x_c, H = x_d - x_c (Blondel and Karplus 1996)
        double F[3], G[3], H[3];
        for (int c = 0; c < 3; ++c) {
            F[c] = X[3 * id[0] + c] - X[3 * id[1] + c];
            G[c] = X[3 * id[1] + c] - X[3 * id[2] + c];
            H[c] = X[3 * id[3] + c] - X[3 * id[2] + c];
        }
        const double A[3] = {F[1] * G[2] - F[2] * G[1], F[2] * G[0] - F[0] * G[2], F[0] * G[1] - F[1] * G[0]};
        const double Bv[3] = {H[1] * G[2] - H[2] * G[1], H[2] * G[0] - H[0] * G[2], H[0] * G[1] - H[1] * G[0]};
        const double AA = A[0] * A[0] + A[1] * A[1] + A[2] * A[2];
        const double BB = Bv[0] * Bv[0] + Bv[1] * Bv[1] + Bv[2] * Bv[2];
        const double GG = G[0] * G[0] + G[1] * G[1] + G[2] * G[2];
        const double nG = sqrt(GG);
        // cos phi = A.B/(|A||B|); sin phi from (B x A).G/|G| (cis = 0)
        const double AxB_G = (Bv[1] * A[2] - Bv[2] * A[1]) * G[0] + (Bv[2] * A[0] - Bv[0] * A[2]) * G[1] +
                             (Bv[0] * A[1] - Bv[1] * A[0]) * G[2];
        const double phi = atan2(AxB_G / nG, A[0] * Bv[0] + A[1] * Bv[1] + A[2] * Bv[2]);
        double s1, c1, s2, c2, s3, c3, s4, c4;
        sincos(phi, &s1, &c1);
        sincos(2.0 * phi, &s2, &c2);
        sincos(3.0 * phi, &s3, &c3);
        sincos(4.0 * phi, &s4, &c4);
        e = 0.5 * (V[0] * (1.0 + c1) + V[1] * (1.0 - c2) + V[2] * (1.0 + c3) + V[3] * (1.0 - c4));
        const double de = 0.5 * (-V[0] * s1 + 2.0 * V[1] * s2 - 3.0 * V[2] * s3 + 4.0 * V[3] * s4);
        const double FG = F[0] * G[0] + F[1] * G[1] + F[2] * G[2];
        const double HG = H[0] * G[0] + H[1] * G[1] + H[2] * G[2];
        double* o = FB + 6 * (size_t)L.n_bonds + 9 * (size_t)L.n_angles + 12 * (size_t)k;
        for (int c = 0; c < 3; ++c) {
            const double ga = -nG / AA * A[c];
            const double gd = nG / BB * Bv[c];
            const double gb = nG / AA * A[c] + FG / (AA * nG) * A[c] - HG / (BB * nG) * Bv[c];
            const double gc = HG / (BB * nG) * Bv[c] - FG / (AA * nG) * A[c] - nG / BB * Bv[c];
            o[c] = de * ga;
            o[3 + c] = de * gb;
            o[6 + c] = de * gc;
            o[9 + c] = de * gd;
        }
    }
    return e;
}

// Pairwise sum of v[0 .. N): halves are added, then quarters, and so on.
template <int N>
__device__ __forceinline__ double tree_sum(double (&v)[N]) {
#pragma unroll
    for (int s = N / 2; s > 0; s >>= 1)
#pragma unroll
        for (int w = 0; w < s; ++w) v[w] += v[w + s];
    return v[0];
}

// Energy of a workgroup: pairwise sum over its threads (`tid`), stored by
// thread 0.  The same order for any number of wavefronts that hold the same
// values: across wavefronts first, then across lanes.
template <int WAVES>
__device__ __forceinline__ void block_energy_store(double e, double* out, int tid) {
    if (WAVES > 1) {
        __shared__ double red[WAVES][64];
        red[tid >> 6][tid & 63] = e;
        __syncthreads();
        if (tid >= 64) return;
        double v[WAVES];
#pragma unroll
        for (int w = 0; w < WAVES; ++w) v[w] = red[w][tid];
        e = tree_sum<WAVES>(v);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) e += __shfl_xor(e, o, 64);
    if (tid == 0) *out = e;
}

// Bonded terms of one evaluation (any precision mode: always FP64): the first
// workgroups of the pair kernel's grid (map_bonded), which evaluates them in
// the shadow of the pair sums instead of in a launch of its own.
template <int THREADS>
__device__ __forceinline__ void bonded_block(const Args& a, int wg, int prec) {
    const int2 m = at<int2>(a.ws, a.L.off_map_bonded)[wg];
    if (m.y == 0 && threadIdx.x == 0) ctl_at(a, m.x)->fin_ticket = 0u;
    if (!eval_active(a, m.x, prec)) return;
    const SysInfo si = sys_info(a)[m.x];
    const double* X = eval_coords(a, m.x, si);
    // a lane's terms (four at most) are added pairwise too
    double even = 0.0, odd = 0.0;
#pragma unroll 1
    for (int t = (int)threadIdx.x; t < kBondedPerBlock; t += THREADS) {
        const double e = bonded_term(a, X, si, m.y * kBondedPerBlock + t);
        if (t / THREADS & 1) odd += e;
        else even += e;
    }
    block_energy_store<THREADS / 64>(even + odd, at<double>(a.ws, a.L.off_eb) + si.eb0 + m.y, threadIdx.x);
}

// Pairs of i-atom i with the atoms J0 .. J0 + 63 of a tile that count: bit jj is
// set if J0 + jj > i and the pair is not excluded.  excl: the atom's near
// exclusions (bit b: i + 1 + b), far: its far ones in this tile (bit jj).
// Returned rotated so that bit s belongs to step s of lane `lane`.
__device__ __forceinline__ uint64_t step_mask(int i, int J0, uint64_t excl, uint64_t far, int lane) {
    const int sh = i + 1 - J0;               // bit of atom i + 1
    uint64_t after, ex;
    if (sh <= 0) {
        after = ~0ull;
        ex = -sh < 64 ? excl >> (-sh) : 0ull;
    } else {
        after = sh < 64 ? ~0ull << sh : 0ull;
        ex = sh < 64 ? excl << sh : 0ull;
    }
    const uint64_t keep = after & ~ex & ~far;
    return (keep >> lane) | (keep << ((64 - lane) & 63));
}

// ---------------------------------------------------------------- FP32 pairs

// i-atoms of one lane: high halves of the coordinates and the per-atom
// factors stay in registers; the low halves live in LDS (s_ilo) because only
// the rare close-pair path reads them.
template <int IPL>
struct IAtoms32 {
    float xh[IPL], yh[IPL], zh[IPL];
    float a12[IPL], b6[IPL], q[IPL];     // 12 c12, 6 c6, q^
};

// A pair closer than sqrt(kCorrR2) by the high halves: redo the displacement
// with both halves in FP64.  Below sqrt(kClashR2) the whole pair is evaluated
// in FP64 (clash energies reach 1e15 kcal/mol at the start of a minimization)
// and the FP32 path is switched off for it by r2 = inf.
template <int IPL>
__device__ __forceinline__ void close_pair32(const IAtoms32<IPL>& I, int k, float4 pj, float4 lo, float4 ilo,
                                          float2 cj, float& dx, float& dy, float& dz, float& r2,
                                          double& gx, double& gy, double& gz, double& e64,
                                          float& fjx, float& fjy, float& fjz) {
    const double ddx = ((double)pj.x - (double)I.xh[k]) + ((double)lo.x - (double)ilo.x);
    const double ddy = ((double)pj.y - (double)I.yh[k]) + ((double)lo.y - (double)ilo.y);
    const double ddz = ((double)pj.z - (double)I.zh[k]) + ((double)lo.z - (double)ilo.z);
    const double rr = ddx * ddx + ddy * ddy + ddz * ddz;
    if (rr < kClashR2) {
        const double rinv = 1.0 / sqrt(rr);
        const double rinv2 = rinv * rinv;
        const double rinv6 = rinv2 * rinv2 * rinv2;
        const double A = (double)I.a12[k] * (double)cj.x, B = (double)I.b6[k] * (double)cj.y;
        const double u = A * rinv6 - B;
        const double ec = (double)I.q[k] * (double)pj.w * rinv;
        e64 += (u - B) * rinv6 * (1.0 / 12.0) + ec;
        const double f = (u * rinv6 + ec) * rinv2;
        gx += f * ddx; gy += f * ddy; gz += f * ddz;
        fjx -= (float)(f * ddx); fjy -= (float)(f * ddy); fjz -= (float)(f * ddz);
        r2 = __builtin_inff();
    } else {
        dx = (float)ddx; dy = (float)ddy; dz = (float)ddz;
        r2 = __fmaf_rn(dz, dz, __fmaf_rn(dy, dy, dx * dx));
    }
}

// The 64 steps of a j-tile: at step s lane l takes atom (l + s) mod 64.
// MASKED: only the pairs of `keep` (step_mask) count; the mask is made once per
// tile (20 chains of 1,500 atoms: 62.7 us, 71 with the exclusions looked up in
// every step; two words of 32 steps with a loop each are as fast there and cost
// 50,000 atoms 1.5 %).
template <int IPL, bool MASKED, bool CHECK>
__device__ __forceinline__ void tile32(const float4* __restrict__ s_xq, const float2* __restrict__ s_c,
                                       const float4* __restrict__ s_lo, const float4* __restrict__ s_ilo,
                                       int lane, int il0, const uint64_t (&keep)[IPL],
                                       const IAtoms32<IPL>& I, float (&fx)[IPL], float (&fy)[IPL],
                                       float (&fz)[IPL], double (&gx)[IPL], double (&gy)[IPL],
                                       double (&gz)[IPL], float& fjx, float& fjy, float& fjz,
                                       float& elj, float& ec32, double& e64) {
    // The loop without checks is fetched best when it starts 16 bytes into a
    // 32-byte block: 50,000 atoms take 848 us there and 857-861 us at the other
    // multiples of 8 bytes.
    if (!MASKED && !CHECK) asm volatile(".p2align 5\n.rept 4\ns_nop 0\n.endr");
    int64_t bits[IPL];                           // the next step's in the sign bit
    if (MASKED) {
#pragma unroll
        for (int k = 0; k < IPL; ++k) bits[k] = (int64_t)__brevll(keep[k]);
    }
#pragma unroll kUnroll32<IPL>
    for (int s = 0; s < kTile; ++s) {
        const int js = lane + s;
        const float4 pj = s_xq[js];
        const float2 cj = s_c[js];
#pragma unroll
        for (int k = 0; k < IPL; ++k) {
            float dx = pj.x - I.xh[k];
            float dy = pj.y - I.yh[k];
            float dz = pj.z - I.zh[k];
            float r2 = __fmaf_rn(dz, dz, __fmaf_rn(dy, dy, dx * dx));
            if (MASKED) {
                r2 = bits[k] < 0 ? r2 : __builtin_inff();
                bits[k] <<= 1;
            }
            if (CHECK && r2 < kCorrR2)
                close_pair32<IPL>(I, k, pj, s_lo[js], s_ilo[il0 + k * 64], cj, dx, dy, dz, r2, gx[k], gy[k],
                                  gz[k], e64, fjx, fjy, fjz);
            const float rinv = __builtin_amdgcn_rsqf(r2);
            const float rinv2 = rinv * rinv;
            const float rinv6 = rinv2 * rinv2 * rinv2;
            const float A = I.a12[k] * cj.x;
            const float B = I.b6[k] * cj.y;
            const float ec = I.q[k] * pj.w * rinv;
            const float u = __fmaf_rn(A, rinv6, -B);
            const float f = __fmaf_rn(u, rinv6, ec) * rinv2;
            elj = __fmaf_rn(u - B, rinv6, elj);
            ec32 += ec;
            fx[k] = __fmaf_rn(f, dx, fx[k]);
            fy[k] = __fmaf_rn(f, dy, fy[k]);
            fz[k] = __fmaf_rn(f, dz, fz[k]);
            fjx = __fmaf_rn(-f, dx, fjx);
            fjy = __fmaf_rn(-f, dy, fjy);
            fjz = __fmaf_rn(-f, dz, fjz);
        }
        fjx = rotate_down(fjx);
        fjy = rotate_down(fjy);
        fjz = rotate_down(fjz);
    }
}

// op over a wavefront, every lane receives it: through the LDS crossbar, which
// leaves the vector units to the other wavefronts, or (REGS) by register
// exchanges (permlane swaps, DPP rotations of 16 lanes), which are sooner done
// (50,000 atoms: 858 us against 889; 512 atoms: 12.6 against 12.1).
template <bool REGS, typename OP>
__device__ __forceinline__ float wave_reducef(float v, OP op) {
    if (!REGS) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v = op(v, __shfl_xor(v, o, 64));
        return v;
    }
    const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = op(__uint_as_float(h[0]), __uint_as_float(h[1]));
    const auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = op(__uint_as_float(q[0]), __uint_as_float(q[1]));
    v = op(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x128, 0xF, 0xF, true)));   // row_ror:8
    v = op(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x124, 0xF, 0xF, true)));
    v = op(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x122, 0xF, 0xF, true)));
    return op(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x121, 0xF, 0xF, true)));
}
template <bool REGS>
__device__ __forceinline__ float wave_minf(float v) {
    return wave_reducef<REGS>(v, [](float a, float b) { return fminf(a, b); });
}
template <bool REGS>
__device__ __forceinline__ float wave_maxf(float v) {
    return wave_reducef<REGS>(v, [](float a, float b) { return fmaxf(a, b); });
}

__device__ __forceinline__ void split(double v, float& hi, float& lo) {
    hi = (float)v;
    lo = (float)(v - (double)hi);
}

// HAS_FAR: the context has excluded pairs more than kExclWindow apart (the
// kernel then checks every tile for a far-exclusion mask; the check costs a
// few registers, so contexts without such pairs run the kernel without it).
// Occupancy floor: with two atoms per lane the kernel fits 168 VGPRs, three
// wavefronts per SIMD, but the compiler's own choice exceeds that by a few
// registers and loses a wavefront.  (The far-exclusion variant would spill
// at 168 and keeps the compiler's choice.)
template <int IPL, bool HAS_FAR>
constexpr int kPair32MinWaves = IPL == 2 && !HAS_FAR ? 3 : 1;

template <int WAVES, int IPL, bool HAS_FAR>
__global__ void __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(kPair32MinWaves<IPL, HAS_FAR>)))
k_pair32(Args a) {
    const Layout& L = a.L;
    const int wg = (int)blockIdx.x - L.n_bonded_blocks;
    if (wg < 0) {
        if (a.bonded) bonded_block<64 * WAVES>(a, blockIdx.x, 1);
        return;
    }
    const ChunkInfo ch = at<ChunkInfo>(a.ws, L.off_chunks[0])[wg];
    if (!eval_active(a, ch.sys, 1)) return;
    const SysInfo si = sys_info(a)[ch.sys];
    const double* X = eval_coords(a, ch.sys, si);
    constexpr int B = 64 * WAVES * IPL;
    const int lane = threadIdx.x & 63;
    const int wave = IPL == 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : threadIdx.x >> 6;
    const int n = si.n, aoff = si.aoff;
    const float* C12 = at<float>(a.ws, L.off_c12);
    const float* C6 = at<float>(a.ws, L.off_c6);
    const float* Q = at<float>(a.ws, L.off_q);
    const uint64_t* EX = at<uint64_t>(a.ws, L.off_excl);
    const int32_t* FU = at<int32_t>(a.ws, L.off_far_unit);
    const uint64_t* FM = at<uint64_t>(a.ws, L.off_far_mask);
    const int I0 = ch.row * B;

    IAtoms32<IPL> I;
    double gx[IPL], gy[IPL], gz[IPL];
    __shared__ float4 s_ilo[B];
    const int il0 = wave * 64 * IPL + lane;     // local index of this lane's first i-atom
    const int i0 = I0 + il0;
    // Coordinates relative to the I-block's first atom: the FP32 displacement
    // of a pair beyond the double-single range then carries the rounding of
    // the pair's own distance, not of the atoms' distance from the origin
    // (for a 1e-3 A step of a relaxed 10,000-atom chain this cuts the rounding
    // noise of the energy difference about 60-fold).
    // (kept in LDS for the j-tile staging: registers are at their limit)
    __shared__ double s_org[3];
    double org[3];
    // With one i-atom per lane, where chunks are one or a few tiles, the first
    // j-tile's atoms are on their way while the i-atoms are set up (with two
    // the registers are at their limit).
    constexpr bool kAhead = IPL == 1;
    constexpr bool kRegs = WAVES * IPL == 1;     // systems too small to fill the SIMDs
    double pj[3];
    float qj = 0.0f;
    float2 cj = make_float2(0.0f, 0.0f);
    auto load_tile = [&](int t) {
        const int j = t * kTile + (int)threadIdx.x;
        load_pos(X, j - aoff, n, pj);
        qj = Q[j];
        cj = make_float2(C12[j], C6[j]);
    };
    if (kAhead && threadIdx.x < kTile) load_tile(ch.t_begin);
    load_pos(X, I0 - aoff, n, org);
    if (threadIdx.x == 0) { s_org[0] = org[0]; s_org[1] = org[1]; s_org[2] = org[2]; }
#pragma unroll
    for (int k = 0; k < IPL; ++k) {
        const int i = i0 + k * 64;
        double p[3];
        load_pos(X, i - aoff, n, p);
        float4 lo;
        split(p[0] - org[0], I.xh[k], lo.x);
        split(p[1] - org[1], I.yh[k], lo.y);
        split(p[2] - org[2], I.zh[k], lo.z);
        lo.w = 0.0f;
        s_ilo[il0 + k * 64] = lo;
        I.a12[k] = 12.0f * C12[i]; I.b6[k] = 6.0f * C6[i]; I.q[k] = Q[i];
        gx[k] = gy[k] = gz[k] = 0.0;
    }
    // bounding box of this wave's i-atoms: a j-tile whose box is farther than
    // sqrt(kCorrR2) cannot hold a close pair, so it runs the unchecked body
    float ib[6];
    ib[0] = ib[3] = I.xh[0];
    ib[1] = ib[4] = I.yh[0];
    ib[2] = ib[5] = I.zh[0];
#pragma unroll
    for (int k = 1; k < IPL; ++k) {
        ib[0] = fminf(ib[0], I.xh[k]); ib[3] = fmaxf(ib[3], I.xh[k]);
        ib[1] = fminf(ib[1], I.yh[k]); ib[4] = fmaxf(ib[4], I.yh[k]);
        ib[2] = fminf(ib[2], I.zh[k]); ib[5] = fmaxf(ib[5], I.zh[k]);
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) { ib[c] = wave_minf<kRegs>(ib[c]); ib[3 + c] = wave_maxf<kRegs>(ib[3 + c]); }
    __shared__ float s_jbox[6];
    __shared__ float4 s_xq[2 * kTile];
    __shared__ float2 s_c[2 * kTile];
    __shared__ float4 s_lo[2 * kTile];
    __shared__ float s_fj[WAVES][3][kTile];
    double e64 = 0.0;
    const int t_masked_end = (I0 + B) / kTile + 1;   // tiles that can hold j <= i or exclusions
    for (int t = ch.t_begin; t < ch.t_end; ++t) {
        const int J0 = t * kTile;
        __syncthreads();
        if (threadIdx.x < kTile) {
            if (!kAhead || t > ch.t_begin) load_tile(t);
            float4 h, l;
            split(pj[0] - s_org[0], h.x, l.x);
            split(pj[1] - s_org[1], h.y, l.y);
            split(pj[2] - s_org[2], h.z, l.z);
            h.w = qj;
            l.w = 0.0f;
            const float2 c = cj;
            s_xq[threadIdx.x] = h; s_xq[threadIdx.x + kTile] = h;
            s_lo[threadIdx.x] = l; s_lo[threadIdx.x + kTile] = l;
            s_c[threadIdx.x] = c;  s_c[threadIdx.x + kTile] = c;
            const float b0 = wave_minf<kRegs>(h.x), b1 = wave_minf<kRegs>(h.y), b2 = wave_minf<kRegs>(h.z);
            const float b3 = wave_maxf<kRegs>(h.x), b4 = wave_maxf<kRegs>(h.y), b5 = wave_maxf<kRegs>(h.z);
            if (threadIdx.x == 0) {
                s_jbox[0] = b0; s_jbox[1] = b1; s_jbox[2] = b2;
                s_jbox[3] = b3; s_jbox[4] = b4; s_jbox[5] = b5;
            }
        }
        __syncthreads();
        float fx[IPL], fy[IPL], fz[IPL];
#pragma unroll
        for (int k = 0; k < IPL; ++k) fx[k] = fy[k] = fz[k] = 0.0f;
        float fjx = 0.0f, fjy = 0.0f, fjz = 0.0f, elj = 0.0f, ec32 = 0.0f;
        const float gxb = fmaxf(0.0f, fmaxf(s_jbox[0] - ib[3], ib[0] - s_jbox[3]));
        const float gyb = fmaxf(0.0f, fmaxf(s_jbox[1] - ib[4], ib[1] - s_jbox[4]));
        const float gzb = fmaxf(0.0f, fmaxf(s_jbox[2] - ib[5], ib[2] - s_jbox[5]));
        const bool far = gxb * gxb + gyb * gyb + gzb * gzb >= kCorrR2;
        const int fu = HAS_FAR ? FU[ch.unit + t - ch.t_begin] : -1;
        uint64_t keep[IPL];
        if ((HAS_FAR && fu >= 0) || t < t_masked_end) {
#pragma unroll
            for (int k = 0; k < IPL; ++k)
                keep[k] = step_mask(i0 + k * 64, J0, EX[i0 + k * 64],
                                    HAS_FAR && fu >= 0 ? FM[(size_t)fu * B + il0 + k * 64] : 0ull, lane);
            tile32<IPL, true, true>(s_xq, s_c, s_lo, s_ilo, lane, il0, keep, I, fx, fy, fz, gx, gy, gz, fjx, fjy, fjz,
                                    elj, ec32, e64);
        } else if (!far)
            tile32<IPL, false, true>(s_xq, s_c, s_lo, s_ilo, lane, il0, keep, I, fx, fy, fz, gx, gy, gz, fjx, fjy, fjz,
                                     elj, ec32, e64);
        else
            tile32<IPL, false, false>(s_xq, s_c, s_lo, s_ilo, lane, il0, keep, I, fx, fy, fz, gx, gy, gz, fjx, fjy, fjz,
                                      elj, ec32, e64);
#pragma unroll
        for (int k = 0; k < IPL; ++k) { gx[k] += fx[k]; gy[k] += fy[k]; gz[k] += fz[k]; }
        e64 += (double)elj * (1.0 / 12.0) + (double)ec32;
        s_fj[wave][0][lane] = fjx;
        s_fj[wave][1][lane] = fjy;
        s_fj[wave][2][lane] = fjz;
        __syncthreads();
        if (wave == 0) {
            double sx = 0.0, sy = 0.0, sz = 0.0;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                sx += (double)s_fj[w][0][lane];
                sy += (double)s_fj[w][1][lane];
                sz += (double)s_fj[w][2][lane];
            }
            float* pj = at<float>(a.ws, L.off_pj) + ((size_t)(ch.j_row + t - ch.t_begin) * kTile + lane) * 3;
            pj[0] = (float)sx; pj[1] = (float)sy; pj[2] = (float)sz;
        }
    }
    // FP32 mode stores its partial sums in single precision (they are FP32
    // tile sums already); the finalize adds them up in FP64
    float* pi = at<float>(a.ws, L.off_pi) + (size_t)ch.slot * B * 3;
#pragma unroll
    for (int k = 0; k < IPL; ++k) {
        const int il = wave * 64 * IPL + k * 64 + lane;
        pi[3 * il] = (float)gx[k]; pi[3 * il + 1] = (float)gy[k]; pi[3 * il + 2] = (float)gz[k];
    }
    block_energy_store<WAVES>(e64, at<double>(a.ws, L.off_ep) + ch.slot, threadIdx.x);
}

// ---------------------------------------------------------------- FP64 pairs

// 1/sqrt(x) for finite x > 0: v_rsq_f64, then y (1 + e/2 + 3e^2/8) with
// e = 1 - x y^2 (the error of the estimate enters cubed), the same
// arithmetic rsqrt uses for such x.  For 0 and infinity e is not a number and
// so is the result; SPECIAL keeps rsqrt's values there (e = 1 leaves the
// estimate's infinity or 0).  Unmasked tiles hold no excluded pair, so x is
// finite and positive, or 0 for coincident atoms, whose energy is not finite
// either way.
template <bool SPECIAL>
__device__ __forceinline__ double rsqrt_step(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    double e = fma(-x * y, y, 1.0);
    if (SPECIAL) e = fmin(e, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}

// Steps [s0, s1) of a j-tile (multiples of kPartSteps): at step s lane l takes
// atom (l + s) mod 64, whose values are read one step ahead.  MASKED: only the
// pairs of `keep` (step_mask) count.
// (whole parts unrolled: a taken branch costs as much as seven operations)
template <bool MASKED>
constexpr int kUnroll64 = MASKED ? 2 : kPartSteps;

template <int IPL, bool MASKED>
__device__ __forceinline__ void tile64(const double4* __restrict__ s_xq, const double2* __restrict__ s_c, int lane,
                                       int s0, int s1, const double (&xi)[IPL], const double (&yi)[IPL],
                                       const double (&zi)[IPL], const double (&a12i)[IPL],
                                       const double (&b6i)[IPL], const double (&qi)[IPL],
                                       const uint64_t (&keep)[IPL],
                                       double (&gx)[IPL], double (&gy)[IPL], double (&gz)[IPL],
                                       double& fjx, double& fjy, double& fjz, double& elj, double& ecs) {
    double4 pn = s_xq[lane + s0];
    double2 cn = s_c[lane + s0];
    // the loop without masks starts in the middle of a 64-byte block: 0.4 % less
    // per evaluation than where the compiler puts it, in the median over 512 to
    // 60,000 atoms (512 atoms: 14.94 us against 15.00; at 50,000, 1,345 and 1,346,
    // the 1-2 % between runs hide it)
    if (!MASKED) asm volatile(".p2align 6\n.rept 8\ns_nop 0\n.endr");
#pragma unroll 1
    for (int sp = s0; sp < s1; sp += kPartSteps) {
        int bits[IPL];                       // mask of the part's steps, the next one in the sign bit
        if (MASKED) {
#pragma unroll
            for (int k = 0; k < IPL; ++k) bits[k] = (int)__brev((unsigned)(keep[k] >> sp));
        }
        const double4* xq = s_xq + lane + sp;
        const double2* xc = s_c + lane + sp;
#pragma unroll kUnroll64<MASKED>
        for (int s = 0; s < kPartSteps; ++s) {
            const double4 pj = pn;
            const double2 cj = cn;
            pn = xq[s + 1];
            cn = xc[s + 1];
#pragma unroll
            for (int k = 0; k < IPL; ++k) {
                const double dx = pj.x - xi[k], dy = pj.y - yi[k], dz = pj.z - zi[k];
                const double r2 = dx * dx + dy * dy + dz * dz;
                double rinv = rsqrt_step<MASKED>(r2);
                if (MASKED) {
                    rinv = bits[k] < 0 ? rinv : 0.0;
                    bits[k] <<= 1;
                }
                const double rinv2 = rinv * rinv;
                const double rinv6 = rinv2 * rinv2 * rinv2;
                const double A = a12i[k] * cj.x;
                const double B = b6i[k] * cj.y;
                const double ec = qi[k] * pj.w * rinv;
                const double u = fma(A, rinv6, -B);
                const double f = fma(u, rinv6, ec) * rinv2;
                elj = fma(u - B, rinv6, elj);
                ecs += ec;
                gx[k] += f * dx; gy[k] += f * dy; gz[k] += f * dz;
                fjx -= f * dx; fjy -= f * dy; fjz -= f * dz;
            }
            fjx = rotate_down(fjx);
            fjy = rotate_down(fjy);
            fjz = rotate_down(fjz);
        }
    }
}

// LDS of one chunk: the j-tile twice in a row, and the j-side sums of several
// wavefronts.
template <int WAVES>
struct Chunk64Lds {
    double4 xq[2 * kTile];
    double2 c[2 * kTile];
    double fj[WAVES > 1 ? WAVES : 1][3][kTile];
};
// Orders the LDS accesses of the WAVES wavefronts that share a chunk.
template <int WAVES>
__device__ __forceinline__ void chunk_sync() {
    if (WAVES > 1) {
        __syncthreads();
    } else {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

// One chunk by WAVES wavefronts of IPL i-atoms per lane; `tid` numbers their
// threads.
template <int WAVES, int IPL>
__device__ __forceinline__ void pair64_chunk(const Args& a, int id, int tid, Chunk64Lds<WAVES>& lds) {
    const Layout& L = a.L;
    const ChunkInfo ch = at<ChunkInfo>(a.ws, L.off_chunks[1])[id];
    if (!eval_active(a, ch.sys, 0)) return;
    const SysInfo si = sys_info(a)[ch.sys];
    const double* X = eval_coords(a, ch.sys, si);
    constexpr int B = 64 * WAVES * IPL;
    const int lane = tid & 63, wave = tid >> 6;
    const int n = si.n, aoff = si.aoff;
    const double* C12 = at<double>(a.ws, L.off_c12d);
    const double* C6 = at<double>(a.ws, L.off_c6d);
    const double* Q = at<double>(a.ws, L.off_qd);
    const uint64_t* EX = at<uint64_t>(a.ws, L.off_excl);
    const int32_t* FU = at<int32_t>(a.ws, L.off_far_unit);
    const uint64_t* FM = at<uint64_t>(a.ws, L.off_far_mask);
    const int I0 = ch.row * B;
    const int i0 = I0 + wave * 64 * IPL + lane;

    // the j-tile's atom of this thread, loaded ahead of its use
    double pj[3], qj = 0.0, c12j = 0.0, c6j = 0.0;
    auto load_tile = [&](int t) {
        const int j = t * kTile + tid;
        load_pos(X, j - aoff, n, pj);
        qj = Q[j]; c12j = C12[j]; c6j = C6[j];
    };
    const bool any_far = L.n_far_units > 0;
    double xi[IPL], yi[IPL], zi[IPL], a12i[IPL], b6i[IPL], qi[IPL], gx[IPL], gy[IPL], gz[IPL];
    double elj = 0.0, ecs = 0.0;     // 12 x Lennard-Jones energy, Coulomb energy
    double4* s_xq = lds.xq;
    double2* s_c = lds.c;
    const int t_masked_end = (I0 + B) / kTile + 1;
    if (tid < kTile) load_tile(ch.t_begin);
#pragma unroll
    for (int k = 0; k < IPL; ++k) {
        const int i = i0 + k * 64;
        double p[3];
        load_pos(X, i - aoff, n, p);
        xi[k] = p[0]; yi[k] = p[1]; zi[k] = p[2];
        a12i[k] = 12.0 * C12[i]; b6i[k] = 6.0 * C6[i]; qi[k] = Q[i];
        gx[k] = gy[k] = gz[k] = 0.0;
    }
    for (int t = ch.t_begin; t < ch.t_end; ++t) {
        const int J0 = t * kTile;
        chunk_sync<WAVES>();
        if (tid < kTile) {
            const double4 h = make_double4(pj[0], pj[1], pj[2], qj);
            const double2 c = make_double2(c12j, c6j);
            s_xq[tid] = h; s_xq[tid + kTile] = h;
            s_c[tid] = c;  s_c[tid + kTile] = c;
            if (t + 1 < ch.t_end) load_tile(t + 1);
        }
        chunk_sync<WAVES>();
        const int s0 = t == ch.t_begin ? ch.steps & 0xff : 0;
        const int s1 = t == ch.t_end - 1 ? ch.steps >> 8 : kTile;
        double fjx = 0.0, fjy = 0.0, fjz = 0.0;
        const int fu = any_far ? FU[ch.unit + t - ch.t_begin] : -1;
        uint64_t keep[IPL];
        if (fu >= 0 || t < t_masked_end) {
#pragma unroll
            for (int k = 0; k < IPL; ++k)
                keep[k] = step_mask(i0 + k * 64, J0, EX[i0 + k * 64],
                                    fu >= 0 ? FM[(size_t)fu * B + i0 - I0 + k * 64] : 0ull, lane);
            tile64<IPL, true>(s_xq, s_c, lane, s0, s1, xi, yi, zi, a12i, b6i, qi, keep, gx, gy, gz, fjx, fjy, fjz, elj,
                              ecs);
        } else {
            tile64<IPL, false>(s_xq, s_c, lane, s0, s1, xi, yi, zi, a12i, b6i, qi, keep, gx, gy, gz, fjx, fjy, fjz,
                               elj, ecs);
        }
        // lane l now holds the sum for atom (l + s1) mod 64 of the tile
        if (WAVES > 1) {
            lds.fj[wave][0][lane] = fjx;
            lds.fj[wave][1][lane] = fjy;
            lds.fj[wave][2][lane] = fjz;
            chunk_sync<WAVES>();
            if (wave == 0) {
                fjx = fjy = fjz = 0.0;
#pragma unroll
                for (int w = 0; w < WAVES; ++w) { fjx += lds.fj[w][0][lane]; fjy += lds.fj[w][1][lane]; fjz += lds.fj[w][2][lane]; }
            }
        }
        if (wave == 0) {
            double* o = at<double>(a.ws, L.off_pj) +
                        ((size_t)(ch.j_row + t - ch.t_begin) * kTile + ((lane + s1) & (kTile - 1))) * 3;
            o[0] = fjx; o[1] = fjy; o[2] = fjz;
        }
    }
    double* pi = at<double>(a.ws, L.off_pi) + (size_t)ch.slot * B * 3;
#pragma unroll
    for (int k = 0; k < IPL; ++k) {
        const int il = wave * 64 * IPL + k * 64 + lane;
        pi[3 * il] = gx[k]; pi[3 * il + 1] = gy[k]; pi[3 * il + 2] = gz[k];
    }
    block_energy_store<WAVES>(elj * (1.0 / 12.0) + ecs, at<double>(a.ws, L.off_ep) + ch.slot, tid);
}

// A workgroup holds four chunks of one wavefront each, or one chunk of several
// wavefronts (fewer workgroups to launch and to send home in cycles without an
// FP64 evaluation).  The kernel walks the chunks with a grid stride: in FP32
// mode (and in cycles without an evaluation) its workgroups only check and
// exit, and a capped grid keeps that cheap.
__host__ __device__ constexpr int group64(int waves) { return waves == 1 ? 4 : 1; }
constexpr int kPair64Grid = 4096;

template <int WAVES, int IPL>
__global__ void __launch_bounds__(64 * WAVES * group64(WAVES)) k_pair64(Args a) {
    // a single system's activity check for the whole launch; in a batch each
    // chunk checks its own system
    if (a.L.n_sys == 1 && !eval_active(a, 0, 0)) return;
    constexpr int G = group64(WAVES);
    __shared__ Chunk64Lds<WAVES> lds[G];
    const int sub = G > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
    const int tid = G > 1 ? threadIdx.x & 63 : threadIdx.x;
    const int nb = a.L.n_bonded_blocks;
    if ((int)blockIdx.x < nb) {
        if (a.bonded) bonded_block<64 * WAVES * G>(a, blockIdx.x, 0);
        return;
    }
    for (int id = ((int)blockIdx.x - nb) * G + sub; id < a.L.n_chunks[1]; id += ((int)gridDim.x - nb) * G)
        pair64_chunk<WAVES, IPL>(a, id, tid, lds[sub]);
}

// ------------------------------------------------------------- host launch
// Tile configurations (index = Layout::cfg): I-block of B = 64 * waves * ipl
// atoms.  Both precisions use the same B (the same rows and units); each
// walks its own chunk table.
#define FF_PAIR_CASE(ID)                                                                           \
    case ID: {                                                                                     \
        constexpr TileConfig T = kTileConfigs[ID];                                                 \
        if (prec && a.L.n_far_units > 0)                                                              \
            hipLaunchKernelGGL((k_pair32<T.waves32, T.ipl32, true>), dim3(nb + grid), dim3(64 * T.waves32), 0, s, a); \
        else if (prec)                                                                                \
            hipLaunchKernelGGL((k_pair32<T.waves32, T.ipl32, false>), dim3(nb + grid), dim3(64 * T.waves32), 0, s, a); \
        else {                                                                                         \
            constexpr int G = group64(T.waves64);                                                      \
            const int wgs = (grid + G - 1) / G;                                                        \
            hipLaunchKernelGGL((k_pair64<T.waves64, T.ipl64>), dim3(nb + (wgs < kPair64Grid ? wgs : kPair64Grid)), \
                               dim3(64 * T.waves64 * G), 0, s, a);                                     \
        }                                                                                              \
        break;                                                                                     \
    }

hipError_t launch_pair(const Args& a, int prec, hipStream_t s) {
    const int grid = a.L.n_chunks[prec ? 0 : 1], nb = a.L.n_bonded_blocks;
    switch (a.L.cfg) {
        FF_PAIR_CASE(0)
        FF_PAIR_CASE(1)
        FF_PAIR_CASE(2)
        FF_PAIR_CASE(3)
        FF_PAIR_CASE(4)
        FF_PAIR_CASE(5)
        FF_PAIR_CASE(6)
        FF_PAIR_CASE(7)
        FF_PAIR_CASE(8)
        FF_PAIR_CASE(9)
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace ff
