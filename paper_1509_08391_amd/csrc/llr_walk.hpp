// llr_walk.hpp -- the sequential part of a heatbath pass under the per-link
// constraint: the walk of one wavefront over a chain's class links, shared by the
// class-pass kernel (llr_sweep.hip, candidates staged from memory) and the
// chain-resident sweep (llr_chain.hip, candidates in LDS).
#pragma once
#include "llr_internal.hpp"
#include "llr_link.hpp"

namespace llr {

constexpr long long kLinkNone = (long long)0x8000000000000000ull;   // no free candidate within the cap

// ---------------------------------------------------------------------------
// Heatbath class pass under the per-link constraint (Sec. 2.4: the energy
// restriction imposed when each new angle is generated).  The links of the
// class are taken one after another in half-index order, each from its
// conditional restricted to the values that keep the running energy in
// [lo, hi], and the energy is carried from link to link.  Links of one class
// share no plaquette, so only that energy couples them.  Per link: the first
// of the class heatbath's own attempts (same counters) that passes the
// sampler test AND keeps E inside; if none of the 64 does, the exact arc
// sampler (attempts 64..127 of the counter's attempt field): on
// x = |X| in [acos u_hi, acos u_lo], where the window on cos X is [u_lo, u_hi],
// exp(k cos x) lies under exp(k u_hi - lam (x - x_a)) with
// lam = k min(sin x_a, (u_hi - u_lo)/(x_b - x_a)), since the secant slope of
// cos from x_a is the mean of sin over [x_a, x], smallest at an end of the
// arc; x comes from that truncated exponential, is kept with probability
// exp(k (cos x - u_hi) + lam (x - x_a)), and its sign is a fair bit.
//
// Before the walk every class link has its free heatbath candidate (the first
// attempt passing the sampler test), that candidate's Delta E in the walk's fixed
// point, and its staples and old angle.  The candidate is the constrained draw
// whenever it keeps E inside.  The walk (one wavefront per chain) scans the
// candidates in order, 1024 at a time: prefix sums of Delta E, and per lane their
// least and greatest value on the way, give the first lane and then the first
// link whose candidate leaves [lo, hi].  Re-draws come in clusters, so 8 attempts
// of that link and of the 7 after it are computed at once (none depends on the
// running energy) and those of the 8 whose candidate leaves the window, given the
// draws before, are resolved one after another by ballots; the lowest accepted
// attempt that stays inside wins.  A link with none among the 8 takes all 64
// attempts and then the arc sampler, one per lane.  The rest of the step is
// checked again with its sums shifted by the change of Delta E.  E is carried
// exactly in fixed point (12 bits finer than the class sums), so the result does
// not depend on the scan's blocking.
//
// What bounds it is the latency of this chain of dependent steps on one
// wavefront.  Cycles of a pass of L = 8 (2048 links, window 123, FP32; mean over
// chains): 16 k for scanning, 0.9 k per batch of 8 links (6.5 batches), 0.6 k per
// re-drawn link (12.6) and 2 k per link that 8 attempts did not settle (3.2).
// Redrawing one link at a time with a full check of the step after each took
// 110 us per pass of 32 such chains (the slowest chain's time), this 60.
// ---------------------------------------------------------------------------
constexpr int kWalkPer = 16;             // links per lane per scan step (1024 per step)

__device__ __forceinline__ long long fx_bound(double v) {
    return v > 4.0e18 ? 4000000000000000000ll : (v < -4.0e18 ? -4000000000000000000ll : (long long)v);
}

// Attempt `att` of class link h: whether the sampler accepts it, the angle and
// its fixed-point Delta E (the walk's window is the caller's test).
template <typename T>
struct LinkTry {
    bool acc;
    T t_new;
    long long d;
};
template <typename T>
__device__ __forceinline__ LinkTry<T> link_try(const LatDev& L, uint32_t h, int att, T C, T S, T t_old, int colour,
                                               int kind, uint32_t sweep, uint32_t c3, uint32_t k0, uint32_t k1,
                                               double a) {
    using M = Math<T>;
    T so, co;
    M::sincos_rad(t_old, &so, &co);
    const T eps_old = fms2(C, co, S, so);
    const T R = M::sqrt_(fma2(C, C, S, S));
    const T kap = (T)a * R;
    const T ak = M::abs_(kap);
    T q, rm1, kg2;
    vm_constants(ak, q, rm1, kg2);
    const uint32_t c1base = ctr1_word(0, (uint32_t)colour, (uint32_t)kind, (uint32_t)L.lat_id);
    const uint4 w = philox10(make_uint4(h, c1base | (uint32_t)(att >> 1), sweep, c3), k0, k1);
    T ch, sh, dE;
    LinkTry<T> r;
    r.acc = vm_try((att & 1) ? w.z : w.x, (att & 1) ? w.w : w.y, q, rm1, kg2, ch, sh);
    r.acc = ak == T(0) ? att == 0 : r.acc;   // no coupling: attempt 0, uniform
    hb_new_angle(ch, sh, C, S, R, kap, eps_old, r.t_new, dE);
    r.d = r.acc ? link_fixed(dE, L) : 0;
    return r;
}

// Re-draw class link h with the running sum Ssum before it (whole wavefront;
// staples and old angle from LDS).  Returns the link's fixed-point Delta E
// on every lane and stores its new angle.
template <typename T, typename Store>
__device__ __forceinline__ long long link_redraw(const LatDev& L, Store&& store, uint32_t h, T C, T S, T t_old, int colour,
                                                 int kind, uint32_t sweep, uint32_t c3, uint32_t k0, uint32_t k1,
                                                 double a, double fxw, double Erun, double lo, double hi,
                                                 long long Ssum, long long lo_fx, long long hi_fx, unsigned& arcs) {
    using M = Math<T>;
    const int lane = threadIdx.x & 63;
    T so, co;
    M::sincos_rad(t_old, &so, &co);
    const T eps_old = fms2(C, co, S, so);
    const T R = M::sqrt_(fma2(C, C, S, S));
    const T kap = (T)a * R;
    const T ak = kap < T(0) ? -kap : kap;
    T q, rm1, kg2;
    vm_constants(ak, q, rm1, kg2);
    // the sampler's attempts, attempt j = lane on this lane
    const uint32_t c1base = ctr1_word(0, (uint32_t)colour, (uint32_t)kind, (uint32_t)L.lat_id);
    const uint4 w = philox10(make_uint4(h, c1base | (uint32_t)(lane >> 1), sweep, c3), k0, k1);
    T ch = T(1), sh = T(0);
    bool acc;
    if (ak == T(0)) {
        acc = lane == 0;
        M::sincos_halfpi_w(w.x, &sh, &ch);
    } else {
        acc = (lane & 1) ? vm_attempt(w.z, w.w, q, rm1, kg2, ch, sh) : vm_attempt(w.x, w.y, q, rm1, kg2, ch, sh);
    }
    T t_c = t_old, dE_c = T(0);
    long long d_c = 0;
    bool ok = false;
    if (acc) {
        hb_new_angle(ch, sh, C, S, R, kap, eps_old, t_c, dE_c);
        d_c = link_fixed(dE_c, L);
        ok = Ssum + d_c >= lo_fx && Ssum + d_c <= hi_fx;
    }
    const unsigned long long m1 = __ballot(ok);
    if (m1) {
        const int f = __ffsll((long long)m1) - 1;
        if (lane == f) store(h, t_c);
        return __shfl(d_c, f, 64);
    }
    // exact arc sampler, in FP64 for either state precision
    const double Rd = (double)R, kd = (double)kap, akd = (double)ak, ed = (double)eps_old;
    const double Aw = lo - (Erun - ed), Bw = hi - (Erun - ed);
    double ulo = -1.0, uhi = 1.0;
    if (Rd > 0.0) {
        ulo = fmin(1.0, fmax(-1.0, kd < 0.0 ? -Bw / Rd : Aw / Rd));
        uhi = fmin(1.0, fmax(-1.0, kd < 0.0 ? -Aw / Rd : Bw / Rd));
    }
    const double xa = acos(uhi), xb = acos(ulo), W = xb - xa;
    bool ok2 = false;
    double t2 = 0.0;
    long long d2 = 0;
    if (W > 0.0) {
        const double lam = akd * fmin(sin(xa), (uhi - ulo) / W);
        const uint4 v = philox10(
            make_uint4(h, ctr1_word((uint32_t)(64 + lane), (uint32_t)colour, (uint32_t)kind, (uint32_t)L.lat_id),
                       sweep, c3), k0, k1);
        const double V = (double)M::unif(v.x), U = (double)M::unif(v.y);
        const double Tt = lam * W < 1e-12 ? V * W : -log1p(V * expm1(-lam * W)) / lam;
        const double xx = fmin(xa + Tt, xb);
        if (log(U) <= akd * (cos(xx) - uhi) + lam * Tt) {
            const double X = (v.z >> 31) ? -xx : xx;
            const double sg = kd < 0.0 ? -1.0 : 1.0;
            double sx, cx;
            sincos(X, &sx, &cx);
            const double Cd = (double)C, Sd = (double)S;
            t2 = atan2(sg * (sx * Cd - cx * Sd), sg * (cx * Cd + sx * Sd));
            if (t2 >= 3.14159265358979323846) t2 -= 6.28318530717958647692;
            d2 = __double2ll_rn((sg * Rd * cx - ed) * fxw);
            ok2 = Ssum + d2 >= lo_fx && Ssum + d2 <= hi_fx;
        }
    }
    const unsigned long long m2 = __ballot(ok2);
    if (m2) {
        const int f = __ffsll((long long)m2) - 1;
        if (lane == f) store(h, (T)t2);
        ++arcs;
        return __shfl(d2, f, 64);
    }
    if (lane == 0) store(h, t_old);
    return 0;
}

// One chain's walk over a class: what stays the same from tile to tile, and the
// running sum of Delta E (fixed point, relative to E0).
struct Walk {
    int colour, kind;
    uint32_t sweep, c3, k0, k1;
    double a, E0, lo, hi, fxw, fxwinv;
    long long lo_fx, hi_fx;
    long long Ssum;
    unsigned fixes, arcs;
};
__device__ __forceinline__ Walk walk_begin(const LatDev& L, int colour, int kind, uint32_t sweep, uint32_t c3,
                                           uint32_t k0, uint32_t k1, double a, double E0, double lo, double hi) {
    Walk w{colour, kind, sweep, c3, k0, k1, a, E0, lo, hi, 0.0, 0.0, 0, 0, 0, 0u, 0u};
    w.fxw = L.fx * (double)(1 << kWalkBits);
    w.fxwinv = L.fxinv / (double)(1 << kWalkBits);
    w.lo_fx = fx_bound(ceil((lo - E0) * w.fxw));
    w.hi_fx = fx_bound(floor((hi - E0) * w.fxw));
    return w;
}

// Walk links t0 .. t0 + nt - 1 of the class (one wavefront): sd, sc, ss, st hold
// their candidates' Delta E, staples and old angles in LDS; a re-drawn link's
// angle goes to store(link, angle).
template <typename T, typename Store>
__device__ __forceinline__ void walk_links(const LatDev& L, Walk& w, uint32_t t0, int nt, const long long* sd,
                                           const T* sc, const T* ss, const T* st, Store&& store) {
    const int lane = threadIdx.x & 63;
    int j0 = 0;
    while (j0 < nt) {
        // one step: candidates j0 .. j0 + 1023, lane l owning 16 l .. 16 l + 15;
        // per lane the total of their Delta E and the least and greatest
        // sum on the way
        const int e0 = j0 + kWalkPer * lane, jend = min(j0 + kWalkPer * 64, nt);
        long long loc = 0, mn = 0, mx = 0;
        bool none = false;   // an entry without a free candidate
#pragma unroll
        for (int q = 0; q < kWalkPer; ++q) {
            const long long d = e0 + q < nt ? sd[e0 + q] : 0;
            none |= d == kLinkNone;
            loc += d == kLinkNone ? 0 : d;
            mn = q == 0 || loc < mn ? loc : mn;
            mx = q == 0 || loc > mx ? loc : mx;
        }
        // running sum before this lane's first entry; a re-draw shifts
        // it by the same delta for every later entry of the step
        const long long incl = wave_scan_i64(loc);
        long long base = w.Ssum + incl - loc;
        const long long tot = lane_i64(incl, 63);
        long long shift = 0;
        int pos = j0, lane0 = 0;   // entries before pos, lanes before lane0 are settled
        for (;;) {
            // the first lane, then its first entry from pos on, whose
            // candidate leaves the window
            const unsigned long long ml =
                __ballot(lane >= lane0 && e0 < jend && (none || base + mn < w.lo_fx || base + mx > w.hi_fx));
            if (ml == 0) break;
            const int f = __ffsll((long long)ml) - 1;
            const int ef = j0 + kWalkPer * f + (lane & (kWalkPer - 1));
            const long long df = ef < jend ? sd[ef] : 0;
            const long long pf = row_scan_i64(df == kLinkNone ? 0 : df);
            const long long base_f = lane_i64(base, f);
            const unsigned long long me =
                __ballot(lane < kWalkPer && ef >= pos && ef < jend &&
                         (df == kLinkNone || base_f + pf < w.lo_fx || base_f + pf > w.hi_fx));
            if (me == 0) {
                lane0 = f + 1;
                continue;
            }
            const int qf = __ffsll((long long)me) - 1;
            const int b = j0 + kWalkPer * f + qf;
            long long S = qf ? base_f + lane_i64(pf, qf - 1) : base_f;   // before link b
            // 8 attempts of each of the links b .. b + nb - 1 at once, attempt
            // a of link i on lane 8 i + a: none depends on the running
            // energy.  Re-draws come in clusters, where the energy runs
            // along the window's edge, so the next ones are among these.
            const int nb = min(8, jend - b), li8 = lane >> 3;
            const int eb = b + min(li8, nb - 1);
            const LinkTry<T> t = link_try<T>(L, t0 + (uint32_t)eb, lane & 7, sc[eb], ss[eb], st[eb],
                                             w.colour, w.kind, w.sweep, w.c3, w.k0, w.k1, w.a);
            const long long dc = lane < nb ? sd[b + lane] : 0;
            const long long pc = row_scan_i64(dc == kLinkNone ? 0 : dc);   // candidates' sums, lanes 0..7
            long long delta = 0;
            int won = -1;   // this lane's attempt is its link's draw
            int i = 0;      // link b + i, whose candidate leaves the window
            for (;;) {
                const long long Sn = S + t.d;
                const unsigned long long mi = __ballot(t.acc && li8 == i && Sn >= w.lo_fx && Sn <= w.hi_fx);
                long long d_new;
                if (mi) {
                    const int w = __ffsll((long long)mi) - 1;
                    d_new = lane_i64(t.d, w);
                    won = lane == w ? lane : won;
                } else {
                    d_new = link_redraw<T>(L, store, t0 + (uint32_t)(b + i), sc[b + i], ss[b + i],
                                           st[b + i], w.colour, w.kind, w.sweep, w.c3, w.k0, w.k1, w.a, w.fxw,
                                           w.E0 + (double)S * w.fxwinv, w.lo, w.hi, S, w.lo_fx, w.hi_fx, w.arcs);
                }
                ++w.fixes;
                const long long pi = lane_i64(pc, i);
                delta += d_new - (i ? pi - lane_i64(pc, i - 1) : pi);
                S += d_new;
                // the next of them that leaves it, now that S is known
                const long long Sl = S + (pc - pi);
                const unsigned long long mn2 =
                    __ballot(lane > i && lane < nb && (dc == kLinkNone || Sl < w.lo_fx || Sl > w.hi_fx));
                if (mn2 == 0) break;
                const int i2 = __ffsll((long long)mn2) - 1;
                S += lane_i64(pc, i2 - 1) - pi;
                i = i2;
            }
            if (won >= 0) store(t0 + (uint32_t)eb, t.t_new);
            shift += delta;
            if (lane >= f) base += delta;
            pos = b + nb;
            lane0 = (pos - j0) / kWalkPer;
            if (pos >= jend) break;
        }
        w.Ssum += tot + shift;
        j0 = jend;
    }
}

}  // namespace llr
