// Adjoint (vector-Jacobian product) of the particle sums of Eqs. 2-5 (Fu & Laurendeau,
// Sec. II.B), transposed stretching scheme, written out by hand.  (The classical scheme's
// adjoint is composed from this kernel and the forward kernel on the host side: its pair
// term S.(J Gamma_i) equals the transposed term Gamma_i.(J^T S) with the target strength and
// the stretching seed exchanged.)
//
// One pair (target i, source j, r = x_i - x_j) contributes, for seeds (ub_i, Sb_i) on
// (u_i, dGamma_i/dt), with v = Gamma_j x r, w = Gamma_i x Gamma_j, a = ub_i.v, b = Sb_i.w,
// tau = Gamma_i.v, c = Sb_i.r and weights g, h = g'/s, k = h'/s:
//   dphi/dr        = [(a + b) h + tau c k] r + g ub_i x Gamma_j + h c w + h tau Sb_i
//   xbar_i        += dphi/dr,         xbar_j -= dphi/dr
//   Gammabar_i    += g Gamma_j x Sb_i + h c v
//   Gammabar_j    += g (r x ub_i + Sb_i x Gamma_i) + h c (r x Gamma_i)
//
// Gather form, no atomics: each lane owns one particle p of the "lane set" and loops over the
// "loop set" q, collecting the terms where p is the target (role A: weights gA, hA, kA from the
// source core sigma_q, p's seeds) and where p is the source (role B: gB, hB, kB from sigma_p,
// q's seeds).  With r = x_p - x_q, v = Gamma_q x r, R = r x ub_q, E_p = Sb_p x Gamma_p and
// Z_q = Sb_q x Gamma_q:
//   a = ub_p.v, a' = -Gamma_p.R, b = Gamma_q.E_p, b' = Gamma_p.Z_q, tau = Gamma_p.v,
//   c = Sb_p.r, c' = -Sb_q.r, hcs = hA c + hB c'
//   xbar_p += sum [(a+b) hA + tau c kA + (a'+b') hB + tau c' kB] r        (accumulator SR)
//           + ub_p x sum gA Gamma_q                                         (A)
//           + Gamma_p x sum (gB ub_q + hcs Gamma_q)                          (UW)
//           + sum tau (hA Sb_p - hB Sb_q)                                   (T)
//   Gbar_p += (sum gA Gamma_q) x Sb_p + sum (gB (Z_q - R) + hcs v)           (A, Q)
// Terms that are a per-particle vector times a sum over q are summed first and finished once
// per particle, which is what keeps the pair cost near three forward pairs.  Outside every
// core (decided per tile from bounding boxes) the two roles share one set of point-vortex
// weights; inside, each role takes its own core.  The kernel carries 4 pi (g, h, k) and
// scales by 1/(4 pi) at the end.  Per-particle sums are FP32 tile partials folded into two-sum
// pairs (VPM_F32C) or plain FP64 (VPM_F64).
//
// Bound by VALU issue.  Sets too small to fill the chip well with a particle per lane (below about a
// million) give several lanes to a particle, each taking a slice of every staged tile (split_lp).
#include <hip/hip_runtime.h>

#include "device_math.h"

// The FP64 kernels call their in-core weights (a convergent call), and clang then reports the
// unroll requests of the loops around that call as not honoured.
#pragma clang diagnostic ignored "-Wpass-failed"
#include "vpm_internal.h"

namespace vpm {

namespace {

template <typename T>
using V4 = typename std::conditional<std::is_same<T, float>::value, float4, double4>::type;

// Keeps a value opaque to the optimiser so that work derived from it inside the rare core
// branch is not hoisted into the hot path (emits no instruction).
__device__ __forceinline__ float opaque_b(float v) {
    asm volatile("" : "+v"(v));
    return v;
}
__device__ __forceinline__ double opaque_b(double v) {
    asm volatile("" : "+v"(v));
    return v;
}

// 4 pi (g, h, k) inside the core (s2 < cut); SYM: 1/sigma^2 = RHO_FAR^2 / cut.
template <typename T, bool SYM>
__device__ __forceinline__ void core3(T s2, T isig, T cut, T Gf, T Hf, T Kf, T& g, T& h, T& k) {
    T is, is2;
    if (SYM) {
        is2 = T(Prec<T>::kFarRho2) * rcp_fast(opaque_b(cut));
        is = sqrt_fast(is2);
    } else {
        is = opaque_b(isig);
        is2 = is * is;
    }
    T G, Hn, Kn;
    core_weights3_call(s2, is, is2, Gf, Hf, Kf, G, Hn, Kn);
    g = G;
    h = T(-3) * Hn;
    k = T(15) * Kn;
}

// Accumulator slots: 0-2 SR r, 3-5 A, 6-8 UW, 9-11 Q, and with stretching seeds 12-14 T, or without
// role B 12 sum hA tau (T is then that sum times Sb_p).
template <typename T, int WG, bool RA, bool RB, bool STR, bool SYM>
struct Bwd {
    static constexpr bool kComp = std::is_same<T, float>::value;
    static constexpr int kN = STR ? (RB ? 15 : 13) : 12;

    // Both roles with one set of point-vortex weights, g and h = -3 g / s^2 (so k = -5 h / s^2):
    // q1 = (Gamma_q, .), q2 = ub_q, q3 = Sb_q, q4 = Sb_q x Gamma_q (q3, q4 unused without stretching
    // seeds).  Bound by VALU issue, so by the operations: 68 per pair, R on one chain
    // with Z_q and one sum of tau (Sb_p - Sb_q).  With R and Z_q apart, k a weight of its own
    // and the sums of hA tau and of hB tau Sb_q apart there were 73: 65536 hover particles 8410 us,
    // now 8080, 200000 70.9 and 67.7 ms.
    static __device__ __forceinline__ void far_pair(const V4<T>& q1, const V4<T>& q2, const V4<T>& q3,
                                                    const V4<T>& q4, T rx, T ry, T rz, T rinv2, T g, T h,
                                                    const T (&gp)[3], const T (&up)[3], const T (&sp)[3],
                                                    const T (&ep)[3], T (&acc)[kN]) {
        // v = Gamma_q x r,  R = r x ub_q (below)
        const T vx = q1.y * rz - q1.z * ry;
        const T vy = q1.z * rx - q1.x * rz;
        const T vz = q1.x * ry - q1.y * rx;
        acc[3] += g * q1.x;
        acc[4] += g * q1.y;
        acc[5] += g * q1.z;
        acc[6] += g * q2.x;
        acc[7] += g * q2.y;
        acc[8] += g * q2.z;
        T sr;
        if (STR) {
            // D = Z_q - R, so a' + b' = Gamma_p . D and the Q term is g D + hcc v
            const T Dx = fma(rz, q2.y, fma(-ry, q2.z, q4.x));
            const T Dy = fma(rx, q2.z, fma(-rz, q2.x, q4.y));
            const T Dz = fma(ry, q2.x, fma(-rx, q2.y, q4.z));
            // s_ab = a + b + a' + b' = ub_p.v + Gamma_q.E_p + Gamma_p.D, one FMA chain
            T s_ab = up[0] * vx;
            s_ab = fma(up[1], vy, s_ab);
            s_ab = fma(up[2], vz, s_ab);
            s_ab = fma(q1.x, ep[0], s_ab);
            s_ab = fma(q1.y, ep[1], s_ab);
            s_ab = fma(q1.z, ep[2], s_ab);
            s_ab = fma(gp[0], Dx, s_ab);
            s_ab = fma(gp[1], Dy, s_ab);
            s_ab = fma(gp[2], Dz, s_ab);
            // c + c' = (Sb_p - Sb_q) . r
            const T dx = sp[0] - q3.x, dy = sp[1] - q3.y, dz = sp[2] - q3.z;
            T cc = dx * rx;
            cc = fma(dy, ry, cc);
            cc = fma(dz, rz, cc);
            T tau = gp[0] * vx;
            tau = fma(gp[1], vy, tau);
            tau = fma(gp[2], vz, tau);
            const T hcc = h * cc;
            const T ht = h * tau;
            sr = fma(T(-5) * rinv2, ht * cc, h * s_ab);
            acc[12] += ht * dx;
            acc[13] += ht * dy;
            acc[14] += ht * dz;
            acc[6] += hcc * q1.x;
            acc[7] += hcc * q1.y;
            acc[8] += hcc * q1.z;
            acc[9] += g * Dx;
            acc[10] += g * Dy;
            acc[11] += g * Dz;
            acc[9] += hcc * vx;
            acc[10] += hcc * vy;
            acc[11] += hcc * vz;
        } else {
            const T Rx = ry * q2.z - rz * q2.y;
            const T Ry = rz * q2.x - rx * q2.z;
            const T Rz = rx * q2.y - ry * q2.x;
            T s_ab = up[0] * vx;
            s_ab = fma(up[1], vy, s_ab);
            s_ab = fma(up[2], vz, s_ab);
            s_ab = fma(-gp[0], Rx, s_ab);
            s_ab = fma(-gp[1], Ry, s_ab);
            s_ab = fma(-gp[2], Rz, s_ab);
            sr = h * s_ab;
            acc[9] -= g * Rx;
            acc[10] -= g * Ry;
            acc[11] -= g * Rz;
        }
        acc[0] += sr * rx;
        acc[1] += sr * ry;
        acc[2] += sr * rz;
    }

    // Staged tile: l[0] = (x, y, z, 1/sigma), l[1] = (Gamma, cut), with role B l[2] = ub_q and,
    // with stretching seeds, l[3] = Sb_q, l[4] = Sb_q x Gamma_q.
    static constexpr int kArr = RB ? (STR ? 5 : 3) : 2;

    // This lane's slice of a tile: the particles first, first + step, ...  self: the tile index of
    // the lane's own particle (CHECK).
    template <bool CHECK, bool NEAR>
    static __device__ __forceinline__ void tile(const V4<T> (*l)[WG], int first, int step, int cnt, int self,
                                                const T (&xp)[3], const T (&gp)[3], const T (&up)[3],
                                                const T (&sp)[3], const T (&ep)[3], T isig_p, T cut_p,
                                                T (&acc)[kN]) {
        const V4<T>*l2 = l[RB ? 2 : 0], *l3 = l[kArr == 5 ? 3 : 0], *l4 = l[kArr == 5 ? 4 : 0];
        auto one = [&](int jj) __attribute__((always_inline)) {
            const V4<T> q0 = l[0][jj];  // x_q, 1/sigma_q
            const V4<T> q1 = l[1][jj];  // Gamma_q, cut_q
            const T rx = xp[0] - q0.x, ry = xp[1] - q0.y, rz = xp[2] - q0.z;
            const T s2 = rx * rx + ry * ry + rz * rz;
            const T rinv = rsqrt_fast(s2);
            const T rinv2 = rinv * rinv;
            const T Gf = rinv2 * rinv;
            const T Hf = Gf * rinv2;
            const T Kf = Hf * rinv2;
            T gA = Gf, hA = T(-3) * Hf, kA = T(15) * Kf;
            T gB = gA, hB = hA, kB = kA;
            if (NEAR) {
                const T cutA = SYM ? q1.w + cut_p : q1.w;
                const T cutB = SYM ? cutA : cut_p;
                if (RA && s2 < cutA) core3<T, SYM>(s2, q0.w, cutA, Gf, Hf, Kf, gA, hA, kA);
                if (RB && s2 < cutB) {
                    if (SYM && RA) {  // one symmetric core for both roles
                        gB = gA;
                        hB = hA;
                        kB = kA;
                    } else {
                        core3<T, SYM>(s2, isig_p, cutB, Gf, Hf, Kf, gB, hB, kB);
                    }
                }
            }
            if (CHECK && jj == self) gA = hA = kA = gB = hB = kB = T(0);
            if constexpr (!NEAR && !CHECK && RA && RB) {
                // Outside every core both roles share (g, h, k): add the roles' terms before
                // multiplying by the weights.
                far_pair(q1, l2[jj], STR ? l3[jj] : q1, STR ? l4[jj] : q1, rx, ry, rz, rinv2, gA, hA, gp, up, sp,
                         ep, acc);
            } else {
                pair_general(q1, jj, l2, l3, l4, rx, ry, rz, gA, hA, kA, gB, hB, kB, gp, up, sp, ep, acc);
            }
        };
        if constexpr (kComp) {
            // the whole rounds of the slices first, whose end is the same for every lane: a test per lane and
            // particle cost a sixth of the velocity's adjoint (a million sources, 1000 targets 705 us, now 635)
            const int rounds = cnt / step;
#pragma unroll 2
            for (int i = 0, jj = first; i < rounds; ++i, jj += step) one(jj);
            const int last = first + rounds * step;
            if (last < cnt) one(last);
        } else {
            // (twice the pair's code costs the single-role FP64 kernels a wavefront per SIMD)
#pragma unroll 2
            for (int jj = first; jj < cnt; jj += step) one(jj);
        }
    }

    // Both roles with their own weights (cores, excluded pairs, single-role launches).
    static __device__ __forceinline__ void pair_general(const V4<T>& q1, int jj, const V4<T>* l2, const V4<T>* l3,
                                                        const V4<T>* l4, T rx, T ry, T rz, T gA, T hA, T kA, T gB,
                                                        T hB, T kB, const T (&gp)[3], const T (&up)[3],
                                                        const T (&sp)[3], const T (&ep)[3], T (&acc)[kN]) {
        {
            // v = Gamma_q x r
            const T vx = q1.y * rz - q1.z * ry;
            const T vy = q1.z * rx - q1.x * rz;
            const T vz = q1.x * ry - q1.y * rx;
            T sr = T(0);
            if (RA) {
                const T a = up[0] * vx + up[1] * vy + up[2] * vz;
                sr = a * hA;
                acc[3] += gA * q1.x;
                acc[4] += gA * q1.y;
                acc[5] += gA * q1.z;
            }
            if (RB) {
                const V4<T> q2 = l2[jj];  // ub_q
                // R = r x ub_q
                const T Rx = ry * q2.z - rz * q2.y;
                const T Ry = rz * q2.x - rx * q2.z;
                const T Rz = rx * q2.y - ry * q2.x;
                const T ap = -(gp[0] * Rx + gp[1] * Ry + gp[2] * Rz);
                sr += ap * hB;
                acc[6] += gB * q2.x;
                acc[7] += gB * q2.y;
                acc[8] += gB * q2.z;
                acc[9] -= gB * Rx;
                acc[10] -= gB * Ry;
                acc[11] -= gB * Rz;
            }
            if (STR) {
                const T tau = gp[0] * vx + gp[1] * vy + gp[2] * vz;
                T hcs = T(0);
                if (RA) {
                    const T b = q1.x * ep[0] + q1.y * ep[1] + q1.z * ep[2];
                    const T c = sp[0] * rx + sp[1] * ry + sp[2] * rz;
                    sr += b * hA + tau * c * kA;
                    hcs = hA * c;
                    if constexpr (RB) {
                        const T ht = hA * tau;
                        acc[12] += ht * sp[0];
                        acc[13] += ht * sp[1];
                        acc[14] += ht * sp[2];
                    } else {
                        acc[12] += hA * tau;
                    }
                }
                if constexpr (RB) {
                    const V4<T> q3 = l3[jj];  // Sb_q
                    const V4<T> q4 = l4[jj];  // Z_q = Sb_q x Gamma_q
                    const T bp = gp[0] * q4.x + gp[1] * q4.y + gp[2] * q4.z;
                    const T cp = -(q3.x * rx + q3.y * ry + q3.z * rz);
                    sr += bp * hB + tau * cp * kB;
                    hcs += hB * cp;
                    const T ht = hB * tau;
                    acc[12] -= ht * q3.x;
                    acc[13] -= ht * q3.y;
                    acc[14] -= ht * q3.z;
                    acc[9] += gB * q4.x;
                    acc[10] += gB * q4.y;
                    acc[11] += gB * q4.z;
                }
                acc[6] += hcs * q1.x;
                acc[7] += hcs * q1.y;
                acc[8] += hcs * q1.z;
                acc[9] += hcs * vx;
                acc[10] += hcs * vy;
                acc[11] += hcs * vz;
            }
            acc[0] += sr * rx;
            acc[1] += sr * ry;
            acc[2] += sr * rz;
        }
    }
};

// Workgroup bounding box (v[0..2] min, v[3..5] max) and largest cut (v[6]): a shuffle
// reduction per wavefront, then LDS.  Ends with a barrier; every thread gets the result.
template <typename T>
__device__ __forceinline__ void box_reduce(T (&v)[7], T* scratch) {
    wave_minmax_last(v);
    const int wave = threadIdx.x >> 6;
    const int nwave = (blockDim.x + 63) >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 63) {
#pragma unroll
        for (int c = 0; c < 7; ++c) scratch[wave * 7 + c] = v[c];
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 7; ++c) v[c] = scratch[c];
    for (int w = 1; w < nwave; ++w) {
#pragma unroll
        for (int c = 0; c < 7; ++c) v[c] = c < 3 ? fmin(v[c], scratch[w * 7 + c]) : fmax(v[c], scratch[w * 7 + c]);
    }
}

// One workgroup's lane block blk of a lane set [lb, lb + nl) against the loop set
// [ob, ob + no) (indices into the arrays of a; with a.self both sets are the same range).
// The block holds P = 2^lp particles (lp <= 6, or P = WG): the workgroup's lanes form WG / P
// slices that share each staged tile (lane tid: particle tid mod P, slice tid / P, which takes
// the tile's particles slice, slice + WG / P, ...).  The slices' sums are added in FP64 at the
// end, by shuffles within a wavefront and through LDS across wavefronts, in a fixed order.
template <typename T, int WG, bool RA, bool RB, bool STR, bool SYM>
__device__ __forceinline__ void backward_body(const BwdArgs& a, int64_t blk, int64_t lb, int64_t nl, int64_t ob,
                                              int64_t no, int lp) {
    using B = Bwd<T, WG, RA, RB, STR, SYM>;
    constexpr int kN = B::kN;
    constexpr bool kComp = B::kComp;
    __shared__ V4<T> l[B::kArr][WG];
    __shared__ T box[7 * (WG / 64)];
    // the set bases are folded into the pointers (null pointers stay null)
    auto at = [](const void* q, int64_t base) { return q ? static_cast<const T*>(q) + base : nullptr; };
    const T* __restrict__ xl = at(a.xl, lb);
    const T* __restrict__ gl = at(a.gl, lb);
    const T* __restrict__ sl = at(a.sl, lb);
    const T* __restrict__ ubl = at(a.ubl, lb);
    const T* __restrict__ sbl = at(a.sbl, lb);
    const T* __restrict__ xo = at(a.xo, ob);
    const T* __restrict__ go = at(a.go, ob);
    const T* __restrict__ so = at(a.so, ob);
    const T* __restrict__ ubo = at(a.ubo, ob);
    const T* __restrict__ sbo = at(a.sbo, ob);
    const T far2 = T(Prec<T>::kFarRho2);
    const int tid = threadIdx.x;
    const int np = 1 << lp;
    const int slice = tid >> lp, nslice = WG >> lp;
    const int64_t pb0 = blk << lp;
    const int64_t p = pb0 + (tid & (np - 1));
    const bool valid = p < nl;
    const int64_t pp = valid ? p : pb0;

    T xp[3] = {xl[pp], xl[a.ldl + pp], xl[2 * a.ldl + pp]};
    T gp[3] = {T(0), T(0), T(0)};
    if (RB || STR) {
        gp[0] = gl[pp];
        gp[1] = gl[a.ldl + pp];
        gp[2] = gl[2 * a.ldl + pp];
    }
    T sgp = T(1);
    if (RB || SYM) sgp = sl[pp];
    const T isig_p = T(1) / sgp;
    // this particle's role-B core cut (source rule) or its half of the symmetric cut
    const T cut_p = SYM ? T(0.5) * far2 * sgp * sgp : (RB ? far2 * sgp * sgp : T(0));
    T up[3] = {T(0), T(0), T(0)}, sp[3] = {T(0), T(0), T(0)}, ep[3] = {T(0), T(0), T(0)};
    if (RA) {
        up[0] = ubl[pp];
        up[1] = ubl[a.ldl + pp];
        up[2] = ubl[2 * a.ldl + pp];
        if (STR) {
            sp[0] = sbl[pp];
            sp[1] = sbl[a.ldl + pp];
            sp[2] = sbl[2 * a.ldl + pp];
            ep[0] = sp[1] * gp[2] - sp[2] * gp[1];
            ep[1] = sp[2] * gp[0] - sp[0] * gp[2];
            ep[2] = sp[0] * gp[1] - sp[1] * gp[0];
        }
    }
    // bounding box of this workgroup's lane particles and their largest cut
    T bb[7] = {xp[0], xp[1], xp[2], xp[0], xp[1], xp[2], valid ? cut_p : T(0)};
    box_reduce(bb, box);

    T acc[kN], hi[kN], lo[kN];
#pragma unroll
    for (int c = 0; c < kN; ++c) acc[c] = hi[c] = lo[c] = T(0);

    for (int64_t j0 = 0; j0 < no; j0 += WG) {
        const int cnt = int((no - j0) < WG ? (no - j0) : WG);
        __syncthreads();
        // idle slots (tid >= cnt) read the tile's first particle, which keeps the box exact
        const int64_t jl = j0 + (tid < cnt ? tid : 0);
        // sigma_q is needed when q acts as a source (role A) or for the symmetric rule;
        // Gamma_q when q is a source or carries stretching seeds.
        const T sq = (RA || SYM) ? so[jl] : T(1);
        V4<T> v0, v1;
        v0.x = xo[jl]; v0.y = xo[a.ldo + jl]; v0.z = xo[2 * a.ldo + jl]; v0.w = T(1) / sq;
        if (RA || STR) {
            v1.x = go[jl]; v1.y = go[a.ldo + jl]; v1.z = go[2 * a.ldo + jl];
        } else {
            v1.x = v1.y = v1.z = T(0);
        }
        v1.w = SYM ? T(0.5) * far2 * sq * sq : (RA ? far2 * sq * sq : T(0));
        if (tid < cnt) {
            l[0][tid] = v0;
            l[1][tid] = v1;
            if constexpr (RB) {
                V4<T> v2;
                v2.x = ubo[jl]; v2.y = ubo[a.ldo + jl]; v2.z = ubo[2 * a.ldo + jl]; v2.w = T(0);
                l[2][tid] = v2;
                if constexpr (STR) {
                    V4<T> v3, v4;
                    v3.x = sbo[jl]; v3.y = sbo[a.ldo + jl]; v3.z = sbo[2 * a.ldo + jl]; v3.w = T(0);
                    v4.x = v3.y * v1.z - v3.z * v1.y;
                    v4.y = v3.z * v1.x - v3.x * v1.z;
                    v4.z = v3.x * v1.y - v3.y * v1.x;
                    v4.w = T(0);
                    l[3][tid] = v3;
                    l[4][tid] = v4;
                }
            }
        }
        // tile box and its largest role-A cut; the reduction's barriers also publish the tile
        T tb[7] = {v0.x, v0.y, v0.z, v0.x, v0.y, v0.z, tid < cnt ? v1.w : T(0)};
        box_reduce(tb, box);
        T d2 = T(0);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const T gap = fmax(fmax(tb[c] - bb[3 + c], bb[c] - tb[3 + c]), T(0));
            d2 += gap * gap;
        }
        const T reach = SYM ? tb[6] + bb[6] : fmax(tb[6], bb[6]);
        const bool near = d2 < reach;
        const bool diag = a.self && (j0 < pb0 + np) && (pb0 < j0 + cnt);
        const int own = int(p - j0);  // (read only where diag, when it fits)
        if (diag) {
            if (near) B::template tile<true, true>(l, slice, nslice, cnt, own, xp, gp, up, sp, ep, isig_p,
                                                           cut_p, acc);
            else B::template tile<true, false>(l, slice, nslice, cnt, own, xp, gp, up, sp, ep, isig_p,
                                                           cut_p, acc);
        } else {
            if (near) B::template tile<false, true>(l, slice, nslice, cnt, own, xp, gp, up, sp, ep, isig_p,
                                                           cut_p, acc);
            else B::template tile<false, false>(l, slice, nslice, cnt, own, xp, gp, up, sp, ep, isig_p,
                                                           cut_p, acc);
        }
        // FP32 sums run over at most WG terms between folds (a slice takes WG / nslice per tile),
        // and near tiles, whose terms are large, are folded at once: the gradient's error against
        // FP64 is then a third of what it is with the far tiles' terms added to them (hover wake,
        // 65536 particles: 2.2e-7 and 7.5e-7; 5.0e-7 with a particle per lane and a fold per tile).
        if constexpr (kComp) {
            if (near || ((j0 / WG + 1) & (nslice - 1)) == 0 || j0 + WG >= no) {
#pragma unroll
                for (int c = 0; c < kN; ++c) {
                    T s, e;
                    two_sum(hi[c], acc[c], s, e);
                    hi[c] = s;
                    lo[c] += e;
                    acc[c] = T(0);
                }
            }
        }
    }
    double t[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) t[c] = 0.0;
#pragma unroll
    for (int c = 0; c < kN; ++c) t[c] = kComp ? double(hi[c]) + double(lo[c]) : double(acc[c]);
    if (nslice > 1) {
        // np <= 64: every wavefront holds the same particles.  The tile's LDS carries the other
        // wavefronts' sums to wavefront 0, kPer sums at a time.
        constexpr int kWaves = WG / 64;
        constexpr int kFit = int(sizeof(l) / ((kWaves - 1) * 64 * sizeof(double)));
        constexpr int kPer = kFit < kN ? kFit : kN;
        double(*red)[kPer][64] = reinterpret_cast<double(*)[kPer][64]>(&l[0][0]);
        for (int off = np; off < 64; off <<= 1)
#pragma unroll
            for (int c = 0; c < kN; ++c) t[c] += __shfl_xor(t[c], off, 64);
        const int wave = tid >> 6, lane = tid & 63;
#pragma unroll
        for (int c0 = 0; c0 < kN; c0 += kPer) {
            __syncthreads();
            if (wave > 0) {
#pragma unroll
                for (int c = 0; c < kPer; ++c)
                    if (c0 + c < kN) red[wave - 1][c][lane] = t[c0 + c];
            }
            __syncthreads();
            if (wave == 0) {
#pragma unroll
                for (int w = 0; w < kWaves - 1; ++w)
#pragma unroll
                    for (int c = 0; c < kPer; ++c)
                        if (c0 + c < kN) t[c0 + c] += red[w][c][lane];
            }
        }
    }
    // (nothing follows in a caller's loop that this lane must reach before its next barrier)
    if (tid >= np || !valid) return;
    const double u0 = up[0], u1 = up[1], u2 = up[2];
    const double g0 = gp[0], g1 = gp[1], g2 = gp[2];
    const double s0 = sp[0], s1 = sp[1], s2 = sp[2];
    // xbar = SR + ub_p x A + Gamma_p x UW + T
    double xb[3] = {t[0], t[1], t[2]};
    xb[0] += u1 * t[5] - u2 * t[4] + g1 * t[8] - g2 * t[7];
    xb[1] += u2 * t[3] - u0 * t[5] + g2 * t[6] - g0 * t[8];
    xb[2] += u0 * t[4] - u1 * t[3] + g0 * t[7] - g1 * t[6];
    // Gbar = A x Sb_p + Q
    double gb[3] = {t[9], t[10], t[11]};
    if (STR) {
        xb[0] += RB ? t[12] : t[12] * s0;
        xb[1] += RB ? t[13] : t[12] * s1;
        xb[2] += RB ? t[14] : t[12] * s2;
        gb[0] += t[4] * s2 - t[5] * s1;
        gb[1] += t[5] * s0 - t[3] * s2;
        gb[2] += t[3] * s1 - t[4] * s0;
    }
    T* __restrict__ xo_bar = static_cast<T*>(a.xbar) + lb;
    T* __restrict__ go_bar = a.gbar ? static_cast<T*>(a.gbar) + lb : nullptr;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        T* d = xo_bar + c * a.ldg + p;
        *d = T(double(*d) + kInv4PiD * xb[c]);
    }
    // velocity-only target gradients touch x only; a null gbar drops the strength gradient
    // (the classical scheme's composition discards the target-role part it recomputes)
    if ((RB || STR) && go_bar) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            T* d = go_bar + c * a.ldg + p;
            *d = T(double(*d) + kInv4PiD * gb[c]);
        }
    }
}

// FP32: ask for 4 wavefronts per SIMD (<= 128 VGPRs; no spills at these shapes).  FP64 keeps
// the compiler's choice: its accumulators need twice the registers.
template <typename T, int WG, bool RA, bool RB, bool STR, bool SYM>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(4))) void k_backward_f32(BwdArgs a, int lp) {
    backward_body<T, WG, RA, RB, STR, SYM>(a, blockIdx.x, 0, a.nl, 0, a.no, lp);
}
template <typename T, int WG, bool RA, bool RB, bool STR, bool SYM>
__global__ __launch_bounds__(WG) void k_backward_f64(BwdArgs a, int lp) {
    backward_body<T, WG, RA, RB, STR, SYM>(a, blockIdx.x, 0, a.nl, 0, a.no, lp);
}

// Particles per workgroup (log2; 8 = no split) of a lane set of nl particles over a loop set of no.  In
// units of which a pair takes 80 (VALU instructions in FP32, half as many in FP64): a staged tile takes
// 230 for staging, box reduction, folds and waiting, a workgroup 1200 (FP64 750) for its beginning and
// its sums' end.  kSlots workgroups are resident on the chip (four wavefronts per SIMD); fewer than that run
// each wavefront faster, so x = nl / P / kSlots rounds take 0.6 + 0.4 x or x + 0.1, whichever is more
// (fitted to the times of P = 16 ... 256 at 1000-200000 particles).  The boxes of 256 particles are near
// more tiles than those of 64 (a pair 81), and in FP64, where an in-core pair alone on its SIMD takes 130,
// a block among the loop set lasts at least as long as its pairs with a tile.
// So sets of more than 26000 particles run in blocks of 32, of more than 72000 in blocks of 64, and a
// particle per lane is left to more than 940000 (both roles: 600000 hover particles in blocks of 64 558
// ms, 256 590, FP64 1146 and 1178; two million 5980 and 5770) and to few loop particles, whose tile is less
// work than the workgroup itself (262144 lanes over 2 targets, velocity only: 26 us in blocks of 64, 11;
// FP32 over 128: 49 and 36, FP64 71 and 144).
// A function of the two sizes and the type alone, so that a set gets the same sums in a launch of its own
// and in a queue of many sets; blocks of 4 would take 1000 particles alone from 37 to 23 us but a queue of
// 300 sets of 64-600 from 150 to 490 us.
// Measured (FP32, both roles, hover wake, us per call without and with the split): 1000
// particles 393 / 37, 4999 1686 / 143, 16384 4970 / 659, 65536 17890 / 8080, 200000 83300 / 67700.
constexpr int kSplitLpMin = 4, kSplitLpMax = 6, kNoSplitLp = 8;
constexpr int64_t kSlots = 1024;
__host__ __device__ inline int split_lp(int64_t nl, int64_t no, bool f64) {
    if (no > (1 << 20)) no = 1 << 20;  // (the products fit 64 bits; a million are many tiles already)
    const int64_t tiles = (no + 255) >> 8, first = no < 256 ? no : 256;
    int best = kNoSplitLp;
    int64_t least = 0;
    for (int lp = kNoSplitLp; lp >= kSplitLpMin; --lp) {
        if (lp > kSplitLpMax && lp != kNoSplitLp) continue;
        // in sixteenths of a workgroup, the last one not rounded up
        const int64_t wgs = nl >> (lp - 4), slots = 16 * kSlots;
        const int64_t below = (6 * slots + 4 * wgs) / 10, above = wgs + slots / 10;
        const int64_t rounds = below > above ? below : above;
        // a lane's pairs, of the whole tiles and of the last one
        const int64_t pairs = ((no >> 8) << lp) + ((((no & 255) << lp) + 255) >> 8);
        int64_t cost = rounds * ((f64 ? 750 : 1200) + 230 * tiles + (lp == kNoSplitLp ? 81 : 80) * pairs);
        const int64_t alone = f64 ? slots * 130 * (((first << lp) + 255) >> 8) : 0;
        if (alone > cost) cost = alone;
        if (lp == kNoSplitLp || cost < least) {
            best = lp;
            least = cost;
        }
    }
    return best;
}

// A value equal in every lane, moved to scalar registers.
__device__ __forceinline__ int64_t uniform_i64(int64_t v) {
    const uint32_t lo = uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(v))));
    const uint32_t hi = uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(uint64_t(v) >> 32))));
    return int64_t((uint64_t(hi) << 32) | lo);
}

// Many independent sets in one launch: persistent workgroups pop (set, lane block) items,
// ordered by decreasing cost, from the queue's counter; the lane set of item set b is
// [src_off[b], src_off[b+1]) and the loop set [tgt_off[b], tgt_off[b+1]) (exchanged when
// lane_is_tgt).  Every workgroup leaves once the counter passes the item count.
template <typename T, int WG, bool RA, bool RB, bool STR, bool SYM>
__device__ __forceinline__ void backward_queue(const BwdArgs& a, const BatchQueue& q, int item_lp, int lane_is_tgt) {
    __shared__ int item_s;
    for (;;) {
        if (threadIdx.x == 0) item_s = atomicAdd(q.counter, 1);
        __syncthreads();
        // (uniform, so that the set's ranges and pointers stay in scalar registers)
        const int item = __builtin_amdgcn_readfirstlane(item_s);
        __syncthreads();
        if (item >= q.n_items) break;
        const int set = __builtin_amdgcn_readfirstlane(q.items[item].x);
        const int64_t nth = __builtin_amdgcn_readfirstlane(q.items[item].y);
        const int64_t* lo = lane_is_tgt ? q.tgt_off : q.src_off;
        const int64_t* oo = lane_is_tgt ? q.src_off : q.tgt_off;
        const int64_t lb = uniform_i64(lo[set]), nl = uniform_i64(lo[set + 1]) - lb;
        const int64_t ob = uniform_i64(oo[set]), no = uniform_i64(oo[set + 1]) - ob;
        // the item's particles, in the blocks that a launch for this set alone would have
        const int lp = split_lp(nl, no, std::is_same<T, double>::value);
        const int more = item_lp > lp ? item_lp - lp : 0;
        const int64_t b0 = nth << more;
        for (int k = 0; k < (1 << more) && ((b0 + k) << lp) < nl; ++k)
            backward_body<T, WG, RA, RB, STR, SYM>(a, b0 + k, lb, nl, ob, no, lp);
    }
}
template <typename T, int WG, bool RA, bool RB, bool STR, bool SYM>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(4))) void k_backward_batched_f32(
    BwdArgs a, BatchQueue q, int item_lp, int lane_is_tgt) {
    backward_queue<T, WG, RA, RB, STR, SYM>(a, q, item_lp, lane_is_tgt);
}
template <typename T, int WG, bool RA, bool RB, bool STR, bool SYM>
__global__ __launch_bounds__(WG) void k_backward_batched_f64(BwdArgs a, BatchQueue q, int item_lp, int lane_is_tgt) {
    backward_queue<T, WG, RA, RB, STR, SYM>(a, q, item_lp, lane_is_tgt);
}

template <typename T, int WG, bool RA, bool RB, bool STR, bool SYM>
void launch_k(const BwdArgs& a, hipStream_t st) {
    static_assert(WG == 1 << kNoSplitLp, "without a split a particle per lane");
    const int lp = split_lp(a.nl, a.no, std::is_same<T, double>::value);
    const unsigned grid = unsigned((a.nl + (int64_t(1) << lp) - 1) >> lp);
    if constexpr (std::is_same<T, float>::value)
        hipLaunchKernelGGL((k_backward_f32<T, WG, RA, RB, STR, SYM>), dim3(grid), dim3(WG), 0, st, a, lp);
    else
        hipLaunchKernelGGL((k_backward_f64<T, WG, RA, RB, STR, SYM>), dim3(grid), dim3(WG), 0, st, a, lp);
}

// Persistent launch over a queue (grid <= 0: only report the kernel's resident workgroups
// per CU through *occ).
template <typename T, int WG, bool RA, bool RB, bool STR, bool SYM>
hipError_t launch_kq(int grid, const BwdArgs& a, const BatchQueue& q, int item_lp, int lane_is_tgt, int* occ,
                     hipStream_t st) {
    if (grid <= 0) {
        if constexpr (std::is_same<T, float>::value)
            return hipOccupancyMaxActiveBlocksPerMultiprocessor(
                occ, reinterpret_cast<const void*>(k_backward_batched_f32<T, WG, RA, RB, STR, SYM>), WG, 0);
        else
            return hipOccupancyMaxActiveBlocksPerMultiprocessor(
                occ, reinterpret_cast<const void*>(k_backward_batched_f64<T, WG, RA, RB, STR, SYM>), WG, 0);
    }
    if constexpr (std::is_same<T, float>::value)
        hipLaunchKernelGGL((k_backward_batched_f32<T, WG, RA, RB, STR, SYM>), dim3(grid), dim3(WG), 0, st, a, q,
                           item_lp, lane_is_tgt);
    else
        hipLaunchKernelGGL((k_backward_batched_f64<T, WG, RA, RB, STR, SYM>), dim3(grid), dim3(WG), 0, st, a, q,
                           item_lp, lane_is_tgt);
    return hipGetLastError();
}

template <typename T, int WG, bool RA, bool RB>
hipError_t launch_rs(bool stretch, bool sym, const BwdArgs& a, const BatchQueue* q, int item_lp, int grid,
                     int lane_is_tgt, int* occ, hipStream_t st) {
    if (q) {
        if (stretch) {
            if (sym) return launch_kq<T, WG, RA, RB, true, true>(grid, a, *q, item_lp, lane_is_tgt, occ, st);
            return launch_kq<T, WG, RA, RB, true, false>(grid, a, *q, item_lp, lane_is_tgt, occ, st);
        }
        if (sym) return launch_kq<T, WG, RA, RB, false, true>(grid, a, *q, item_lp, lane_is_tgt, occ, st);
        return launch_kq<T, WG, RA, RB, false, false>(grid, a, *q, item_lp, lane_is_tgt, occ, st);
    }
    if (stretch) {
        if (sym) launch_k<T, WG, RA, RB, true, true>(a, st);
        else launch_k<T, WG, RA, RB, true, false>(a, st);
    } else {
        if (sym) launch_k<T, WG, RA, RB, false, true>(a, st);
        else launch_k<T, WG, RA, RB, false, false>(a, st);
    }
    return hipGetLastError();
}

template <typename T>
hipError_t launch_t(bool ra, bool rb, bool stretch, bool sym, const BwdArgs& a, const BatchQueue* q, int item_lp,
                    int grid, int lane_is_tgt, int* occ, hipStream_t st) {
    if (ra && rb) return launch_rs<T, kBwdWG, true, true>(stretch, sym, a, q, item_lp, grid, lane_is_tgt, occ, st);
    if (ra) return launch_rs<T, kBwdWG, true, false>(stretch, sym, a, q, item_lp, grid, lane_is_tgt, occ, st);
    return launch_rs<T, kBwdWG, false, true>(stretch, sym, a, q, item_lp, grid, lane_is_tgt, occ, st);
}

}  // namespace

int backward_split_lp(int64_t nl, int64_t no, bool f64) { return split_lp(nl, no, f64); }

hipError_t launch_backward(int dtype, bool role_a, bool role_b, bool stretch, bool sym,
                           const BwdArgs& a, hipStream_t st) {
    if (a.nl == 0) return hipSuccess;
    if (!role_a && !role_b) return hipErrorInvalidValue;
    if (dtype == kDtypeF64) return launch_t<double>(role_a, role_b, stretch, sym, a, nullptr, 0, 0, 0, nullptr, st);
    return launch_t<float>(role_a, role_b, stretch, sym, a, nullptr, 0, 0, 0, nullptr, st);
}

hipError_t launch_backward_batched(int dtype, bool role_a, bool role_b, bool stretch, bool sym, const BwdArgs& a,
                                   const BatchQueue& q, int item_lp, int grid, int lane_is_tgt, hipStream_t st) {
    if (!role_a && !role_b) return hipErrorInvalidValue;
    if (dtype == kDtypeF64) return launch_t<double>(role_a, role_b, stretch, sym, a, &q, item_lp, grid, lane_is_tgt, nullptr, st);
    return launch_t<float>(role_a, role_b, stretch, sym, a, &q, item_lp, grid, lane_is_tgt, nullptr, st);
}

int backward_occupancy(int dtype, bool role_a, bool role_b, bool stretch, bool sym) {
    int occ = 0;
    BwdArgs a{};
    BatchQueue q{};
    hipError_t e = dtype == kDtypeF64 ? launch_t<double>(role_a, role_b, stretch, sym, a, &q, 0, 0, 0, &occ, nullptr)
                                      : launch_t<float>(role_a, role_b, stretch, sym, a, &q, 0, 0, 0, &occ, nullptr);
    return e == hipSuccess ? occ : 0;
}

}  // namespace vpm
