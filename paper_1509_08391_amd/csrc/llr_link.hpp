// llr_link.hpp -- device arithmetic of one link, shared by the class-pass
// kernels (llr_sweep.hip) and the chain-resident sweep (llr_chain.hip): the
// von Mises sampler, the heatbath and overrelaxation angles, the fixed-point
// energy change, the multicanonical weight and the plaquette cosine.  Both
// files are compiled without floating-point contraction, so a link's result
// does not depend on the kernel that computes it.
#pragma once
#include "llr_internal.hpp"

namespace llr {

// heatbath pass modes: the public LLR_MODE_* values 0-4, the tuner's timing
// mode, and the candidate pre-pass of the per-link constraint (every link's
// free heatbath candidate written with its Delta E and staples, nothing
// accepted, no counters touched; the walk kernel then decides)
enum { kModeRestricted = 0, kModeApproach = 1, kModeFree = 2, kModeMuca = 3, kModeLink = 4,
       kModeTune = kHbModeTune, kModeLinkPre = 6 };
// instantiations of a heatbath pass: plain, with the restriction per link (the
// class pass then only writes candidates), followed by the class's overrelaxation
enum { kHbPlain = 0, kHbPre = 1, kHbFuseOr = 2 };
// Whether a condition that almost never holds does so on any lane: one compare
// and a scalar branch, where a select would cost every lane an instruction per
// value and a divergent branch the copies of its merge.
__device__ __forceinline__ bool any_lane(bool c) { return __builtin_expect(__ballot(c) != 0ull, 0); }

// Best-Fisher constants in the cancellation-free form: q = (1-rho)/(1+rho),
// r - 1 = (1-rho)^2/(2 rho), kappa (r^2 - 1) with sqrt(r^2-1) = (1-rho^2)/(2 rho).
template <typename T>
__device__ __forceinline__ void vm_constants(T ak, T& q, T& rm1, T& kg2) {
    using M = Math<T>;
    // rho = 2 ak / D with D = tau + sqrt(2 tau); in terms of D:
    // q = (D - 2ak)/(D + 2ak), (1-rho)^2/(2 rho) = (D - 2ak)^2/(4 ak D),
    // (1-rho^2)/(2 rho) = (D - 2ak)(D + 2ak)/(4 ak D)
    const T tau = T(1) + M::sqrt_(T(1) + T(4) * ak * ak);
    const T D = tau + M::sqrt_(T(2) * tau);
    const T dm = D - T(2) * ak, dp = D + T(2) * ak;
    if constexpr (M::f32) {
        // 1/(4 ak D) and 1/dp from one reciprocal of their product
        const T fd = T(4) * ak * D;
        const T t = M::div_(T(1), fd * dp);
        const T r1 = dp * t;
        rm1 = dm * dm * r1;
        const T gg = dm * dp * r1;
        kg2 = ak * gg * gg;
        q = dm * (fd * t);
    } else {
        const T r1 = M::div_(T(1), T(4) * ak * D);
        rm1 = dm * dm * r1;
        const T gg = dm * dp * r1;
        kg2 = ak * gg * gg;
        q = M::div_(dm, dp);
    }
    if (any_lane(!(ak > T(0)))) {   // no coupling: a uniform angle
        if (!(ak > T(0))) {
            q = T(1);
            rm1 = T(1);
            kg2 = T(0);
        }
    }
}

// One sampler attempt from the word pair (wa, wb): accept test of Best &
// Fisher with z = cos(pi V1); (c_, s_) = (cos, q sin)(pi V1 / 2).  Both accept
// tests are always evaluated: on nearly every wavefront some lane needs the
// second.
template <typename T>
__device__ __forceinline__ bool vm_try(uint32_t wa, uint32_t wb, T q, T rm1, T kg2, T& c_, T& s_) {
    using M = Math<T>;
    M::sincos_halfpi_w(wa, &s_, &c_);
    s_ = q * s_;
    const T U2 = M::unif(wb);
    const T cc = M::div_(kg2, M::fma_(T(2) * c_, c_, rm1));   // kappa (r^2 - 1)/(r + z)
    const bool squeeze = M::fma_(cc, T(2) - cc, -U2) > T(0);
    bool full;
    if constexpr (M::f32) {
        // ln(c/U2) + 1 - c >= 0 as c >= U2 e^(c - 1): one transcendental
        full = cc >= U2 * __builtin_amdgcn_exp2f(M::fma_(cc, 1.44269504088896341f, -1.44269504088896341f));
    } else {
        full = M::log_(M::div_(cc, U2)) + T(1) - cc >= T(0);
    }
    return squeeze | full;
}
// The same, writing (ch, sh) only on acceptance.
template <typename T>
__device__ __forceinline__ bool vm_attempt(uint32_t wa, uint32_t wb, T q, T rm1, T kg2, T& ch, T& sh) {
    T c_, s_;
    const bool acc = vm_try(wa, wb, q, rm1, kg2, c_, s_);
    ch = acc ? c_ : ch;
    sh = acc ? s_ : sh;
    return acc;
}
// Attempts 0 and 1 of a link from one Philox call: the first accepted one's
// (ch, sh).  Both are evaluated, since on nearly every wavefront some lane needs
// the second.  A link without coupling takes attempt 0 (its q is 1).
template <typename T>
__device__ __forceinline__ bool vm_first_two(const uint4& w, T ak, T q, T rm1, T kg2, T& ch, T& sh) {
    T c1, s1;
    const bool a0 = vm_try(w.x, w.y, q, rm1, kg2, ch, sh);
    const bool a1 = vm_try(w.z, w.w, q, rm1, kg2, c1, s1);
    const bool keep = a0 | (ak == T(0));
    ch = keep ? ch : c1;
    sh = keep ? sh : s1;
    return keep | a1;
}

// Sum over the wavefront (the order does not matter for integers): DPP row
// shifts and broadcasts instead of twelve cross-lane LDS permutes.
template <int CTRL, int ROWS>
__device__ __forceinline__ long long dpp_add(long long v) {
    const int lo = __builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), CTRL, ROWS, 0xf, false);
    return v + (long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}
// inclusive prefix sums within each row of 16 lanes (row_shr:1, 2, 4, 8)
__device__ __forceinline__ long long row_scan_i64(long long v) {
    v = dpp_add<0x111, 0xf>(v);
    v = dpp_add<0x112, 0xf>(v);
    v = dpp_add<0x114, 0xf>(v);
    return dpp_add<0x118, 0xf>(v);
}
// over the wavefront
__device__ __forceinline__ long long wave_scan_i64(long long v) {
    v = row_scan_i64(v);
    v = dpp_add<0x142, 0xa>(v);    // row_bcast:15 into rows 1 and 3
    return dpp_add<0x143, 0xc>(v); // row_bcast:31 into rows 2 and 3
}
__device__ __forceinline__ long long lane_i64(long long v, int lane) {
    return (long long)(((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(v >> 32), lane) << 32) |
                       (unsigned)__builtin_amdgcn_readlane((int)v, lane));
}
__device__ __forceinline__ long long wave_sum_i64(long long v) { return lane_i64(wave_scan_i64(v), 63); }

// The same for 32-bit values: their 16-bit halves add up without overflow, and
// each step is one instruction with a DPP operand.
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_add32(int v) { return v + __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, false); }
__device__ __forceinline__ int wave_sum_small(int v) {
    v = dpp_add32<0x111, 0xf>(v);
    v = dpp_add32<0x112, 0xf>(v);
    v = dpp_add32<0x114, 0xf>(v);
    v = dpp_add32<0x118, 0xf>(v);
    v = dpp_add32<0x142, 0xa>(v);
    v = dpp_add32<0x143, 0xc>(v);
    return __builtin_amdgcn_readlane(v, 63);
}
__device__ __forceinline__ long long wave_sum_i32(int v) {
    return ((long long)wave_sum_small(v >> 16) << 16) + (long long)wave_sum_small(v & 0xffff);
}

// A link's Delta E in the lattice's fixed point 2^-fxb (FP64 path).  The FP32
// path sums a thread's links at 2^-25 in 32 bits (|Delta E| <= 2 R <= 12 per
// link, at most 4 links per thread) and shifts once: fxb >= 26 for L <= 32.
__device__ __forceinline__ long long to_fixed(double v, const LatDev& L) { return __double2ll_rn(v * L.fx); }

// The per-link walk carries the energy kWalkBits finer than the class sums:
// it adds links into a plain 64-bit sum, so the 13 bits the class sums keep
// for their arrival count are free (|sum| <= 6V 2^(fxb + 12) <= 2^61).  An
// FP32 link's Delta E is the class sums' 2^-25 value shifted, so FP32 energies
// are those of the class-wise passes exactly.
constexpr int kWalkBits = 12;

template <typename T>
__device__ __forceinline__ long long link_fixed(T dE, const LatDev& L) {
    if constexpr (Math<T>::f32) return (long long)__float2int_rn(dE * 33554432.0f) << (L.fxb + kWalkBits - 25);
    else return __double2ll_rn((double)dE * (L.fx * (double)(1 << kWalkBits)));
}

// New angle and local-action change of a heatbath link from the accepted
// half-angle pair (c_, s_) = (cos, q sin)(pi V1 / 2): e^{iX} is
// (c_ + i s_)^2 / nrm, negated for a negative coupling, and
// theta' = arg[e^{iX} (C - i S)].
template <typename T>
__device__ __forceinline__ void hb_new_angle(T c_, T s_, T C, T S, T R, T kap, T eps_old, T& t_new, T& dE) {
    using M = Math<T>;
    T er = fms2(c_, c_, s_, s_), ei = T(2) * c_ * s_;
    const T nrm = fma2(c_, c_, s_, s_);
    if (any_lane(kap < T(0))) {
        er = kap < T(0) ? -er : er;
        ei = kap < T(0) ? -ei : ei;
    }
    T pr = C, pi = -S;
    if (any_lane(R == T(0))) {
        pr = R == T(0) ? T(1) : pr;
        pi = R == T(0) ? T(0) : pi;
    }
    const T zr = fms2(er, pr, ei, pi), zi = fma2(er, pi, ei, pr);
    t_new = M::atan2_(zi, zr);
    if (!M::f32 && t_new >= M::pi()) t_new -= T(2) * M::pi();
    dE = M::div_(R * er, nrm) - eps_old;
}

// The fused pass's version of hb_new_angle: the heatbath angle is not
// stored, only its overrelaxation -2 phi - theta' = -phi - X (mod 2 pi), i.e.
// arg[e^{-iX} (C - i S)] (for vanishing staples, -X), so neither the heatbath
// angle's arctangent nor its sine and cosine are needed; dE as there.
template <typename T>
__device__ __forceinline__ void hb_or_new_angle(T c_, T s_, T C, T S, T R, T kap, T eps_old, T& t_or, T& dE) {
    using M = Math<T>;
    T er = fms2(c_, c_, s_, s_), ei = T(2) * c_ * s_;
    const T nrm = fma2(c_, c_, s_, s_);
    if (any_lane(kap < T(0))) {
        er = kap < T(0) ? -er : er;
        ei = kap < T(0) ? -ei : ei;
    }
    T pr = C, pi = -S;
    if (any_lane(R == T(0))) {
        pr = R == T(0) ? T(1) : pr;
        pi = R == T(0) ? T(0) : pi;
    }
    const T zr = fma2(er, pr, ei, pi), zi = fms2(er, pi, ei, pr);   // (er - i ei)(pr + i pi)
    t_or = M::atan2_(zi, zr);
    if (!M::f32 && t_or >= M::pi()) t_or -= T(2) * M::pi();
    dE = M::div_(R * er, nrm) - eps_old;
}

// Overrelaxation of one link with staple sums (C, S): theta' = -2 phi - theta
// = arg[(C - i S)^2 e^{-i theta}]; a link with vanishing staples is reflected.
// (so, co) = (sin, cos) theta, as sincos_rad gives them.
template <typename T>
__device__ __forceinline__ T or_angle_sc(T t, T so, T co, T C, T S) {
    using M = Math<T>;
    const T ar = fms2(C, C, S, S), ai = T(-2) * C * S;   // (C - iS)^2
    const T zr = fma2(ar, co, ai, so);                   // times (cos - i sin)
    const T zi = fms2(ai, co, ar, so);
    T t_new = M::atan2_(zi, zr);
    if (any_lane(C == T(0) && S == T(0))) t_new = C == T(0) && S == T(0) ? -t : t_new;
    if (!M::f32 && t_new >= M::pi()) t_new -= T(2) * M::pi();
    return t_new;
}

template <typename T>
__device__ __forceinline__ T or_angle(T t, T C, T S) {
    T so, co;
    Math<T>::sincos_rad(t, &so, &co);
    return or_angle_sc(t, so, co, C, S);
}

// ln W(E) = -ln rho~(E) of the multicanonical weight (Sec. 2.6): in interval
// k, -ln rho~(c_k) + a_k (E - c_k); below the first and above the last
// interval the first and last pieces continue, i.e. W = e^{a_0 E + c_1} and
// e^{a_{n-1} E + c_2} with the constants fixed by continuity.
__device__ __forceinline__ double muca_lnw(const LatDev& L, const DevState& s, double E) {
    const double* c = s.cen + L.itv0;
    const double lo = c[0] - 0.5 * L.ds;
    int k = (int)floor((E - lo) / L.ds);
    k = k < 0 ? 0 : (k > L.n_itv - 1 ? L.n_itv - 1 : k);
    return -s.mu_lnrho[L.itv0 + k] + s.a[L.itv0 + k] * (E - c[k]);
}

// ---------------------------------------------------------------------------
// cos of a plaquette angle in FP64 (four link angles in [-pi, pi], so
// |x| <= 4 pi): x = k pi + r with |r| <= pi/2 by Cody and Waite's two-part
// reduction (pi_hi keeps 48 significant bits, so k pi_hi is exact for
// |k| <= 8), cos x = (-1)^k cos r, and cos r by its Taylor series through r^22
// (truncation < 2e-17 on |r| <= pi/2; measured error < 2.5e-16 absolute over
// |x| <= 4 pi).  Fifteen FP64 operations, no branches.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double cos_plaq(double x) {
    const double k = rint(x * 0.31830988618379067);          // 1/pi
    double r = __fma_rn(-k, 0x1.921fb54442d00p+1, x);         // pi_hi
    r = __fma_rn(-k, 0x1.8469898cc5170p-47, r);               // pi - pi_hi
    const double u = r * r;
    double c = -0x1.0ce396db7f853p-70;                        // -1/22!
    c = __fma_rn(c, u, 0x1.e542ba4020225p-62);                //  1/20!
    c = __fma_rn(c, u, -0x1.6827863b97d97p-53);               // -1/18!
    c = __fma_rn(c, u, 0x1.ae7f3e733b81fp-45);                //  1/16!
    c = __fma_rn(c, u, -0x1.93974a8c07c9dp-37);               // -1/14!
    c = __fma_rn(c, u, 0x1.1eed8eff8d898p-29);                //  1/12!
    c = __fma_rn(c, u, -0x1.27e4fb7789f5cp-22);               // -1/10!
    c = __fma_rn(c, u, 0x1.a01a01a01a01ap-16);                //  1/8!
    c = __fma_rn(c, u, -0x1.6c16c16c16c17p-10);               // -1/6!
    c = __fma_rn(c, u, 0x1.5555555555555p-5);                 //  1/4!
    c = __fma_rn(c, u, -0.5);
    c = __fma_rn(c, u, 1.0);
    return ((int)k & 1) ? -c : c;
}

}  // namespace llr
