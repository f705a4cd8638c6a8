// llr_chain.hip -- sweeps of small lattices with the whole chain resident in
// LDS (gfx950): one block owns one chain, loads its 8 colour planes (4V
// angles) once, runs any number of sweeps on them and writes them back.
//
// What bounds the class-pass kernels at these sizes is not work: a class of
// L = 4..8 has 128..2048 links per chain, so a pass is one launch of a few
// blocks whose time is the launch, a dependent chain of loads and the
// per-chain reduction (L = 8 x 512 chains, FP32: 20.3 us per heatbath and
// 10.3 us per overrelaxation pass; L = 4 x 8, FP64: 12 and 8 us), and a sweep
// is 16 of them.  Here a pass is LDS reads, arithmetic and one or two block
// barriers; the class decision needs no atomics and no second plane, because
// the proposals of the running class stay in registers until it is taken.
// The arithmetic per link is that of the class-pass kernels (llr_link.hpp)
// and the class sums are the same integers, so the results are theirs bit
// for bit.  Measured per sweep (class passes before): L = 8 x 512 FP32 300 ->
// 123 us, L = 8 x 32 FP32 ~130 -> 70 us, L = 4 x 8 FP64 133 -> 43 us.
#include <hip/hip_runtime.h>

#include "llr_internal.hpp"
#include "llr_link.hpp"
#include "llr_walk.hpp"

namespace llr {

__device__ __forceinline__ int lanes_below(unsigned long long m) {
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

__device__ __forceinline__ float lane_read(float v, int src) {
    return __int_as_float(__builtin_amdgcn_ds_bpermute(4 * src, __float_as_int(v)));
}
__device__ __forceinline__ double lane_read(double v, int src) {
    const int lo = __builtin_amdgcn_ds_bpermute(4 * src, __double2loint(v));
    const int hi = __builtin_amdgcn_ds_bpermute(4 * src, __double2hiint(v));
    return __hiloint2double(hi, lo);
}

// Per-link constants of the launch: the site's half index and the byte
// offsets of its neighbours' half indices, packed in 16 bits each (a chain's
// plane is at most 16 KB).  Along x0 they depend on the parity of x0, which is
// that of (site parity + s): odd sites step up to another half index, even
// ones down.
struct ChainLink {
    int hb;               // half index, bytes
    int w0;               // low half: step up from an odd x0, high half: down from an even one
    int w[3];             // x1, x2, x3: low half up, high half down
    int s;                // (x1 + x2 + x3) & 1
};
__device__ __forceinline__ int lo16(int v) { return (int)(short)v; }
__device__ __forceinline__ int hi16(int v) { return v >> 16; }
__device__ __forceinline__ int pack16(int lo, int hi) { return (lo & 0xffff) | (hi << 16); }

template <typename T>
__device__ __forceinline__ ChainLink chain_link(const LatDev& L, int h) {
    ChainLink k;
    const uint32_t hh = h < (int)L.V2 ? (uint32_t)h : 0u;   // idle lanes compute link 0 and discard it
    const int esz = (int)sizeof(T);
    const uint32_t r1 = L.hL == 1 ? hh : fdiv(hh, L.mhL);
    const int x0h = (int)(hh - r1 * (uint32_t)L.hL);
    const uint32_t r2 = fdiv(r1, L.mL);
    const uint32_t r3 = fdiv(r2, L.mL);
    const int x[3] = {(int)(r1 - r2 * (uint32_t)L.L), (int)(r2 - r3 * (uint32_t)L.L), (int)r3};
    k.hb = (int)hh * esz;
    k.w0 = pack16((x0h == L.hL - 1 ? 1 - L.hL : 1) * esz, (x0h == 0 ? L.hL - 1 : -1) * esz);
#pragma unroll
    for (int n = 0; n < 3; ++n)
        k.w[n] = pack16((x[n] == L.L - 1 ? -L.hwrap[n + 1] : L.hstr[n + 1]) * esz,
                        (x[n] == 0 ? L.hwrap[n + 1] : -L.hstr[n + 1]) * esz);
    k.s = (x[0] + x[1] + x[2]) & 1;
    return k;
}

template <typename T>
__device__ __forceinline__ T lds_at(const char* base, int off) {
    return *reinterpret_cast<const T*>(base + off);
}

// Staple sums of a link of direction mu (uniform) and parity p: the same terms
// in the same order as staples() of the class-pass kernels.  mu is a run-time
// value: one copy of the code for all directions keeps a sweep's instructions
// (heatbath and overrelaxation) inside the instruction cache, where eight
// specialised passes would evict each other, for two selects per direction.
template <typename T>
__device__ __forceinline__ void chain_staples(const char* lat, int pb, int mu, int p, const ChainLink& k, T& C, T& S) {
    using M = Math<T>;
    const bool odd = ((k.s + p) & 1) != 0;
    const int w0 = odd ? k.w0 & 0xffff : k.w0 & ~0xffff;
    const int up_mu = lo16(mu == 0 ? w0 : (mu == 1 ? k.w[0] : (mu == 2 ? k.w[1] : k.w[2])));
    const int mu_q = (2 * mu + (p ^ 1)) * pb;   // byte offset of the plane of theta_mu on the other parity
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        // the j-th of the directions other than mu, ascending
        const bool hi = j >= mu;
        const int nu = j + (hi ? 1 : 0);
        const int wn = hi ? k.w[j] : (j == 0 ? w0 : k.w[j == 0 ? 0 : j - 1]);
        const int up_nu = lo16(wn), dn_nu = hi16(wn);
        const int nu_p = (2 * nu + p) * pb, nu_q = (2 * nu + (p ^ 1)) * pb;
        const T t_nu_pmu = lds_at<T>(lat, nu_q + k.hb + up_mu);
        const T t_mu_pnu = lds_at<T>(lat, mu_q + k.hb + up_nu);
        const T t_nu_x = lds_at<T>(lat, nu_p + k.hb);
        const T t_nu_pmu_mnu = lds_at<T>(lat, nu_p + k.hb + up_mu + dn_nu);
        const T t_mu_mnu = lds_at<T>(lat, mu_q + k.hb + dn_nu);
        const T t_nu_mnu = lds_at<T>(lat, nu_q + k.hb + dn_nu);
        const T sf = t_nu_pmu - t_mu_pnu - t_nu_x;
        const T sb = t_nu_mnu - t_nu_pmu_mnu - t_mu_mnu;
        T s1, c1, s2, c2;
        M::sincos_rad(sf, &s1, &c1);
        M::sincos_rad(sb, &s2, &c2);
        if (j == 0) {
            C = c1 + c2;
            S = s1 + s2;
        } else {
            C += c1 + c2;
            S += s1 + s2;
        }
    }
}

// The value of lane J of each quad on all four of its lanes (one DPP move per word).
template <int J>
__device__ __forceinline__ float quad_lane(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x55 * J, 0xf, 0xf, false));
}
template <int J>
__device__ __forceinline__ double quad_lane(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x55 * J, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x55 * J, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}

// The same with a link on the four lanes of a quad: lane j = 0..2 takes the two
// staples of the j-th direction, lane 3 the sine and cosine of the link's own
// angle t, and every lane gets all the results; the sums run in the same order.
template <typename T>
__device__ __forceinline__ void quad_staples(const char* lat, int pb, int mu, int p, const ChainLink& k, int q, T t,
                                             T& C, T& S, T& so, T& co) {
    using M = Math<T>;
    const bool odd = ((k.s + p) & 1) != 0;
    const int w0 = odd ? k.w0 & 0xffff : k.w0 & ~0xffff;
    const int up_mu = lo16(mu == 0 ? w0 : (mu == 1 ? k.w[0] : (mu == 2 ? k.w[1] : k.w[2])));
    const int mu_q = (2 * mu + (p ^ 1)) * pb;
    const int j = q < 3 ? q : 2;
    const int nu = j + (j >= mu ? 1 : 0);
    const int wn = nu == 0 ? w0 : (nu == 1 ? k.w[0] : (nu == 2 ? k.w[1] : k.w[2]));
    const int up_nu = lo16(wn), dn_nu = hi16(wn);
    const int nu_p = (2 * nu + p) * pb, nu_q = (2 * nu + (p ^ 1)) * pb;
    const T t_nu_pmu = lds_at<T>(lat, nu_q + k.hb + up_mu);
    const T t_mu_pnu = lds_at<T>(lat, mu_q + k.hb + up_nu);
    const T t_nu_x = lds_at<T>(lat, nu_p + k.hb);
    const T t_nu_pmu_mnu = lds_at<T>(lat, nu_p + k.hb + up_mu + dn_nu);
    const T t_mu_mnu = lds_at<T>(lat, mu_q + k.hb + dn_nu);
    const T t_nu_mnu = lds_at<T>(lat, nu_q + k.hb + dn_nu);
    const T sf = t_nu_pmu - t_mu_pnu - t_nu_x;
    const T sb = t_nu_mnu - t_nu_pmu_mnu - t_mu_mnu;
    T s1, c1, s2, c2;
    M::sincos_rad(q == 3 ? t : sf, &s1, &c1);
    M::sincos_rad(sb, &s2, &c2);
    so = quad_lane<3>(s1);
    co = quad_lane<3>(c1);
    const T c = c1 + c2, z = s1 + s2;
    C = quad_lane<0>(c) + quad_lane<1>(c) + quad_lane<2>(c);
    S = quad_lane<0>(z) + quad_lane<1>(z) + quad_lane<2>(z);
}

// Attempts 2 m_from, ... of the links of one wavefront that rejected the ones
// before (the first two: about 9 %): the pending links are packed into slots and the 64 lanes
// are dealt out among them, G lanes per slot, lane i of a slot taking attempt
// pair m0 + i; the first success in attempt order wins.  One round ends
// nearly every wavefront's tail, with no block barrier.
template <typename T, int LPT>
__device__ __forceinline__ void chain_tail(bool (&got)[LPT], T (&ch)[LPT], T (&sh)[LPT], const T (&ak)[LPT],
                                           const ChainLink (&k)[LPT], int* w_h, T* w_ak, int m_from,
                                           uint32_t c1base, uint32_t sweep, uint32_t c3, uint32_t k0, uint32_t k1) {
    const int lane = threadIdx.x & 63;
    bool open[LPT];
#pragma unroll
    for (int r = 0; r < LPT; ++r) open[r] = !got[r];
    for (;;) {
        int np = 0, slot[LPT];
        bool mine[LPT];   // in this batch of at most 64 slots
#pragma unroll
        for (int r = 0; r < LPT; ++r) {
            const unsigned long long m = __ballot(open[r]);
            slot[r] = np + lanes_below(m);
            mine[r] = open[r] && slot[r] < 64;
            np += (int)__popcll(m);
        }
        if (np == 0) return;
        np = min(np, 64);
        for (int m0 = m_from; np > 0 && m0 < kVmCap / 2;) {
#pragma unroll
            for (int r = 0; r < LPT; ++r)
                if (mine[r] && !got[r]) {
                    w_h[slot[r]] = k[r].hb / (int)sizeof(T);
                    w_ak[slot[r]] = ak[r];
                }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            int lg = np <= 1 ? 5 : 6 - (32 - __clz(np - 1));   // largest 2^lg lanes per slot with np 2^lg <= 64
            lg = min(lg, 4);
            while (m0 + (1 << lg) > kVmCap / 2) --lg;
            const int G = 1 << lg;
            const int j = lane >> lg;
            bool acc = false;
            T che = T(1), she = T(0);
            if (j < np) {
                T q, rm1, kg2;
                vm_constants(w_ak[j], q, rm1, kg2);
                const uint4 w = philox10(make_uint4((uint32_t)w_h[j], c1base | (uint32_t)(m0 + (lane & (G - 1))), sweep,
                                                    c3), k0, k1);
                acc = vm_attempt(w.x, w.y, q, rm1, kg2, che, she);
                if (!acc) acc = vm_attempt(w.z, w.w, q, rm1, kg2, che, she);
            }
            const unsigned long long ok = __ballot(acc);
            np = 0;
#pragma unroll
            for (int r = 0; r < LPT; ++r) {
                const bool ask = mine[r] && !got[r];
                const unsigned gm = ask ? (unsigned)(ok >> (slot[r] << lg)) & ((1u << G) - 1u) : 0u;
                const int src = gm ? (slot[r] << lg) + __ffs((int)gm) - 1 : 0;
                const T c_ = lane_read(che, src), s_ = lane_read(she, src);
                if (gm) {
                    got[r] = true;
                    ch[r] = c_;
                    sh[r] = s_;
                }
                const bool left = ask && !gm;
                const unsigned long long m = __ballot(left);
                slot[r] = np + lanes_below(m);
                np += (int)__popcll(m);
            }
            m0 += G;
            __builtin_amdgcn_wave_barrier();
        }
#pragma unroll
        for (int r = 0; r < LPT; ++r)
            if (mine[r]) open[r] = false;   // accepted, or at the attempt cap (the link keeps its angle)
    }
}

// LPT links per thread, link e of thread tid at half index e NT + tid.  GRP = 4:
// one link per quad of lanes.  A pass of L = 4 is one chain of dependent FP64
// instructions (about 10 cycles each, one wavefront per SIMD), which the quad
// shortens: a lane takes two of the six staples, and two of the link's first eight
// sampler attempts, so that the tail below runs once in 10^4 links.
// Decisions, counters, measurement and recompute are those of the last block
// of a class pass, k_end_sweep and k_energy; every thread takes the class
// decision itself from the block's partial sums, which saves a barrier.
// VAR kHbFuseOr: the interleaved order, each heatbath followed by its class's
// overrelaxation on the same staples.  kHbPre: the restriction per link; the
// class's candidates go to LDS (behind the planes) and, in place, to its plane,
// and the first wavefront walks them.  A launch of one pass waits for the chain
// with most re-draws (L = 8 x 32 FP32: 60 us a pass, the chains' mean 15); here
// each chain goes on to its next pass by itself (534 -> 203 us per sweep).
template <typename T, int LPT, int MAXT, int VAR, int GRP>
__global__ __launch_bounds__(MAXT, GRP == 4 ? 2 : 4) void k_chain(LatTable lt, T* __restrict__ th, DevState s, ChainArgs a) {
    using M = Math<T>;
    constexpr bool FUSED = VAR == kHbFuseOr;
    static_assert(GRP == 1 || (GRP == 4 && LPT == 1 && VAR != kHbPre), "a quad of lanes holds one link");
    extern __shared__ __align__(16) char lat[];   // 8 planes of V/2 angles
    __shared__ long long part[2][MAXT / 64];
    __shared__ int w_h[MAXT / 64][64];
    __shared__ T w_ak[MAXT / 64][64];
    const int g = (int)blockIdx.x, tid = (int)threadIdx.x, NT = (int)blockDim.x;
    const int wid = tid >> 6, lane = tid & 63, nw = NT >> 6;
    const int tl = tid / GRP, NL = NT / GRP;      // a thread's first link, and their stride
    const bool lead = GRP == 1 || tid % GRP == 0;   // the lane that writes and counts a link
    int li = 0;
#pragma unroll 1
    while (li + 1 < lt.n && g >= lt.l[li + 1].chain0) ++li;
    const LatDev& L = lt.l[li];
    const int cl = g - L.chain0;
    const int V2 = (int)L.V2, pb = V2 * (int)sizeof(T);
    const bool idle = a.mode == kModeApproach && s.lat_done[li];
    const uint32_t sweep0 = a.approach ? *s.approach_ctr : *s.sweep_ctr;
    const long long row0 = s.bits_row ? *s.bits_row : 0;
    if (!idle) {
        const uint64_t curw = *reinterpret_cast<const uint64_t*>(s.cur + 8 * g);
        T* chain = th + L.base + (long long)cl * 16ll * (long long)V2;
#pragma unroll 1
        for (int c = 0; c < 8; ++c) {
            const T* src = chain + (size_t)(((curw >> (8 * c)) & 1ull) * 8ull + (uint64_t)c) * V2;
            for (int h = tid; h < V2; h += NT) *reinterpret_cast<T*>(lat + c * pb + h * (int)sizeof(T)) = src[h];
        }
        ChainLink k[LPT];
#pragma unroll
        for (int r = 0; r < LPT; ++r) k[r] = chain_link<T>(L, r * NL + tl);
        const int gi = s.itv[g];
        const double lo = s.lo[gi], hi = s.hi[gi];
        const double afix = a.mode == kModeMuca ? s.mu_b[li] : s.a[gi];
        const uint32_t c3 = (uint32_t)(gi - L.itv0);
        const uint32_t kind = a.approach ? (uint32_t)kApproach : (uint32_t)kSweep;
        const bool b_half = a.order == 2 && cl >= (L.n_chains + 1) / 2;   // staggered: overrelaxation first
        double E = s.E[g];
        double sumE = a.measure_from < a.n_sweeps ? s.sumE[gi] : 0.0;
        unsigned prop = 0, nacc = 0, nfused = 0, bits = 0, fixes = 0, arcs = 0;
        int flip = 0;   // which half of `part` the next reduction uses
        __syncthreads();
#pragma unroll 1
        for (int t = 0; t < a.n_sweeps; ++t) {
            const uint32_t sweep = sweep0 + (uint32_t)t;
            bits = 0;
#pragma unroll 1
            for (int ps = 0; ps < (a.approach || FUSED ? 8 : 16); ++ps) {
                const int colour = ps & 7, mu = colour >> 1, p = colour & 1;
                const bool heat = FUSED || (ps < 8) != b_half;
                char* own = lat + colour * pb;
                T C[LPT], S[LPT], t_old[LPT], so[LPT], co[LPT];
#pragma unroll
                for (int r = 0; r < LPT; ++r) {
                    t_old[r] = lds_at<T>(own, k[r].hb);
                    if constexpr (GRP == 4) quad_staples<T>(lat, pb, mu, p, k[r], tid & 3, t_old[r], C[r], S[r], so[r], co[r]);
                    else chain_staples<T>(lat, pb, mu, p, k[r], C[r], S[r]);
                }
                if (!heat) {
#pragma unroll
                    for (int r = 0; r < LPT; ++r) {
                        T tn;
                        if constexpr (GRP == 4) tn = or_angle_sc(t_old[r], so[r], co[r], C[r], S[r]);
                        else tn = or_angle(t_old[r], C[r], S[r]);
                        // (all staples of the class are of other planes: no barrier before the write)
                        if (lead && r * NL + tl < V2) *reinterpret_cast<T*>(own + k[r].hb) = tn;
                    }
                    __syncthreads();
                    continue;
                }
                const double acoup = a.mode == kModeApproach ? s.b[8 * g + colour] : afix;
                const uint32_t c1base = ctr1_word(0, (uint32_t)colour, kind, (uint32_t)L.lat_id);
                T eps_old[LPT], R[LPT], kap[LPT], ak[LPT], ch[LPT], sh[LPT], t_rej[LPT];
                bool got[LPT];
#pragma unroll
                for (int r = 0; r < LPT; ++r) {
                    if constexpr (GRP == 1) M::sincos_rad(t_old[r], &so[r], &co[r]);
                    eps_old[r] = fms2(C[r], co[r], S[r], so[r]);
                    // rejected class: the old angle, or its overrelaxation in the fused order
                    t_rej[r] = t_old[r];
                    if constexpr (FUSED) t_rej[r] = or_angle_sc(t_old[r], so[r], co[r], C[r], S[r]);
                    R[r] = M::sqrt_(fma2(C[r], C[r], S[r], S[r]));
                    kap[r] = (T)acoup * R[r];
                    ak[r] = kap[r] < T(0) ? -kap[r] : kap[r];
                    ch[r] = T(1);
                    sh[r] = T(0);
                    got[r] = true;
                    if ((r * NL + tl < V2)) {
                        T q, rm1, kg2;
                        vm_constants(ak[r], q, rm1, kg2);
                        if constexpr (GRP == 4) {   // two of the first eight attempts per lane
                            const uint4 w = philox10(make_uint4((uint32_t)(r * NL + tl), c1base | (uint32_t)(tid & 3), sweep,
                                                                c3), a.k0, a.k1);
                            got[r] = vm_first_two(w, ak[r], q, rm1, kg2, ch[r], sh[r]);
                        } else {
                            const uint4 w = philox10(make_uint4((uint32_t)(r * NL + tl), c1base, sweep, c3), a.k0, a.k1);
                            got[r] = vm_first_two(w, ak[r], q, rm1, kg2, ch[r], sh[r]);
                        }
                    }
                }
                if constexpr (GRP == 4) {
                    // the first lane of the quad that accepted
                    const unsigned m = (unsigned)(__ballot(got[0]) >> (lane & ~3)) & 15u;
                    const int src = (lane & ~3) + (m ? __ffs((int)m) - 1 : 0);
                    ch[0] = lane_read(ch[0], src);
                    sh[0] = lane_read(sh[0], src);
                    const bool none = m == 0;
                    got[0] = !(none && lead);   // only the leading lane's values count from here on
                    if (any_lane(none))
                        chain_tail<T, LPT>(got, ch, sh, ak, k, w_h[wid], w_ak[wid], 4, c1base, sweep, c3, a.k0, a.k1);
                } else {
                    chain_tail<T, LPT>(got, ch, sh, ak, k, w_h[wid], w_ak[wid], 1, c1base, sweep, c3, a.k0, a.k1);
                }
                if constexpr (VAR == kHbPre) {
                    long long* sd = reinterpret_cast<long long*>(lat + 8 * pb);
                    T* sc = reinterpret_cast<T*>(sd + V2);
                    T *ss = sc + V2, *st = ss + V2;
#pragma unroll
                    for (int r = 0; r < LPT; ++r) {
                        T tn = t_old[r], dE = T(0);
                        if (got[r]) hb_new_angle(ch[r], sh[r], C[r], S[r], R[r], kap[r], eps_old[r], tn, dE);
                        const int h = r * NL + tl;
                        if (h < V2) {
                            sd[h] = got[r] ? link_fixed(dE, L) : kLinkNone;
                            sc[h] = C[r];
                            ss[h] = S[r];
                            st[h] = t_old[r];
                            *reinterpret_cast<T*>(own + k[r].hb) = tn;
                        }
                    }
                    __syncthreads();
                    if (wid == 0) {
                        Walk w = walk_begin(L, colour, (int)kind, sweep, c3, a.k0, a.k1, afix, E, lo, hi);
                        walk_links<T>(L, w, 0u, V2, sd, sc, ss, st,
                                      [&](uint32_t h, T v) { *reinterpret_cast<T*>(own + h * (uint32_t)sizeof(T)) = v; });
                        if (lane == 0) part[0][0] = w.Ssum;
                        fixes += w.fixes;
                        arcs += w.arcs;
                    }
                    __syncthreads();
                    E += (double)part[0][0] * (L.fxinv / (double)(1 << kWalkBits));
                    prop += 1;
                    nacc += 1;
                    bits |= 1u << colour;
                    continue;   // the next write of part[0][0] follows two more barriers
                }
                T t_new[LPT];
                long long fx = 0;
                int fx32 = 0;
#pragma unroll
                for (int r = 0; r < LPT; ++r) {
                    T dE = T(0);
                    t_new[r] = t_rej[r];
                    if (lead && r * NL + tl < V2 && got[r]) {
                        if constexpr (FUSED) hb_or_new_angle(ch[r], sh[r], C[r], S[r], R[r], kap[r], eps_old[r], t_new[r], dE);
                        else hb_new_angle(ch[r], sh[r], C[r], S[r], R[r], kap[r], eps_old[r], t_new[r], dE);
                    }
                    if constexpr (M::f32) fx32 += __float2int_rn(dE * 33554432.0f);
                    else fx += to_fixed((double)dE, L);
                }
                if constexpr (M::f32) fx = wave_sum_i32(fx32) << (L.fxb - 25);
                else fx = wave_sum_i64(fx);
                if (lane == 0) part[flip][wid] = fx;
                __syncthreads();   // also: every thread has read its staples
                long long total = 0;
                for (int w = 0; w < nw; ++w) total += part[flip][w];
                flip ^= 1;
                const double En = E + (double)total * L.fxinv;
                bool acc;
                if (a.mode == kModeRestricted) {
                    acc = En >= lo && En <= hi;
                } else if (a.mode == kModeApproach) {
                    const double d0 = fmax(0.0, fmax(lo - E, E - hi));
                    const double d1 = fmax(0.0, fmax(lo - En, En - hi));
                    acc = d1 <= d0;
                    if (tid == 0) {
                        const double cen = s.cen[gi];
                        const int sg = cen > En ? 1 : (cen < En ? -1 : 0);
                        const int qq = 8 * g + colour;
                        double eta = s.eta[qq];
                        const int sp = s.sprev[qq];
                        if (sp != 0 && sg != 0) eta = sg == sp ? fmin(0.05, 1.2 * eta) : fmax(1e-6, 0.5 * eta);
                        s.eta[qq] = eta;
                        s.b[qq] = fmin(4.0, fmax(0.0, s.b[qq] + eta * (double)sg));
                        s.sprev[qq] = sg;
                    }
                } else if (a.mode == kModeMuca) {
                    const double lr = muca_lnw(L, s, En) - muca_lnw(L, s, E) - acoup * (En - E);
                    const uint4 w = philox10(make_uint4(c3, ctr1_word(0, (uint32_t)colour, kMuca, (uint32_t)L.lat_id),
                                                        sweep, 0u), a.k0, a.k1);
                    acc = lr >= 0.0 || ((double)w.x + 0.5) * 0x1p-32 < exp(lr);
                } else {
                    acc = true;   // free
                }
                prop += 1;
                if (acc) {
                    E = En;
                    bits |= 1u << colour;
                    nacc += 1;
                    if constexpr (FUSED) nfused += 1;
                }
                if (acc || FUSED) {
#pragma unroll
                    for (int r = 0; r < LPT; ++r)
                        if (lead && r * NL + tl < V2) *reinterpret_cast<T*>(own + k[r].hb) = acc ? t_new[r] : t_rej[r];
                }
                __syncthreads();
            }
            const int jt = a.j0 + t;   // position in the recompute period
            if (a.every > 0 && ((jt + 1) % a.every == 0 || jt == a.last)) {
                // E = sum of the plaquette cosines in the lattice's fixed point
                long long fx = 0;
                int bad = 0;
                for (int i = tid; i < 2 * V2; i += NT) {
                    const int p = i >= V2 ? 1 : 0;
                    const ChainLink q = chain_link<T>(L, i - p * V2);
                    const bool odd = ((q.s + p) & 1) != 0;
                    const int up[4] = {odd ? lo16(q.w0) : 0, lo16(q.w[0]), lo16(q.w[1]), lo16(q.w[2])};
                    double own[4];
#pragma unroll
                    for (int m = 0; m < 4; ++m) own[m] = (double)lds_at<T>(lat, (2 * m + p) * pb + q.hb);
#pragma unroll
                    for (int m = 0; m < 4; ++m)
#pragma unroll
                        for (int n = m + 1; n < 4; ++n) {
                            const double t_nu_pmu = (double)lds_at<T>(lat, (2 * n + (p ^ 1)) * pb + q.hb + up[m]);
                            const double t_mu_pnu = (double)lds_at<T>(lat, (2 * m + (p ^ 1)) * pb + q.hb + up[n]);
                            const double ang = own[m] + t_nu_pmu - t_mu_pnu - own[n];
                            bad |= !(fabs(ang) < INFINITY);
                            fx += __double2ll_rn(cos_plaq(ang) * L.fx);
                        }
                }
                fx = wave_sum_i64(fx);
                if (lane == 0) part[flip][wid] = fx;
                const int anybad = __syncthreads_or(bad);
                long long total = 0;
                for (int w = 0; w < nw; ++w) total += part[flip][w];
                flip ^= 1;
                const double En = (double)total * L.fxinv;
                if (tid == 0) {
                    uint32_t f = anybad ? (uint32_t)kHealthNonFinite : 0u;
                    const double bound = (sizeof(T) == 4 ? 1e-5 : 1e-9) * 12.0 * (double)L.V2;
                    const double d = fabs(En - E);
                    if (a.check & kCheckDrift) {
                        s.drift[g] = fmax(s.drift[g], d);
                        if (!(d <= bound)) f |= kHealthDrift;
                    }
                    if ((a.check & kCheckInterval) && !(En >= lo - bound && En <= hi + bound)) f |= kHealthOutside;
                    if (f) atomicOr(s.health + g, f);
                }
                E = En;
            }
            if (tid == 0) {
                if (t >= a.measure_from) sumE += E;
                if (a.E_hist) a.E_hist[(size_t)t * lt.n_chains + g] = E;
                if (a.end_sweep) {
                    // the launch's first sweep takes what single class passes before it left
                    const uint16_t b16 = (uint16_t)(bits | (t == 0 ? s.bits[g] : 0u) | (a.approach ? 0u : 0xff00u));
                    const long long row = row0 + t;
                    if (s.bits_log && row < s.bits_rows_max) s.bits_log[row * lt.n_chains + g] = b16;
                    s.bits_last[g] = b16;
                    if (a.bits_hist) a.bits_hist[(size_t)t * lt.n_chains + g] = b16;
                } else {
                    s.bits[g] |= (uint16_t)bits;   // k_end_sweep follows the replica exchange
                }
            }
        }
        __syncthreads();
#pragma unroll 1
        for (int c = 0; c < 8; ++c) {
            T* dst = chain + (size_t)(((curw >> (8 * c)) & 1ull) * 8ull + (uint64_t)c) * V2;
            for (int h = tid; h < V2; h += NT) dst[h] = *reinterpret_cast<const T*>(lat + c * pb + h * (int)sizeof(T));
        }
        if (tid == 0) {
            s.E[g] = E;
            if (a.measure_from < a.n_sweeps) s.sumE[gi] = sumE;
            s.hb_prop[g] += prop;
            s.hb_acc[g] += nacc;
            s.fu_acc[g] += nfused;
            if (a.end_sweep) s.bits[g] = 0;
            if constexpr (VAR == kHbPre) {
                s.link_fix[g] += fixes;
                s.link_arc[g] += arcs;
            }
        }
    }
    if (idle && a.end_sweep && tid == 0) {
        const uint16_t first = s.bits[g];
        for (int t = 0; t < a.n_sweeps; ++t)
            if (s.bits_log && row0 + t < s.bits_rows_max) s.bits_log[(row0 + t) * lt.n_chains + g] = t == 0 ? first : 0;
        s.bits_last[g] = a.n_sweeps == 1 ? first : 0;
        s.bits[g] = 0;
    }
    if (a.end_sweep && tid == 0) {
        // the block that arrives last advances the counters every block has read
        if (atomicAdd(s.arrive, 1u) == (uint32_t)lt.n_chains - 1u) {
            if (a.approach) *s.approach_ctr = sweep0 + (uint32_t)a.n_sweeps;
            else *s.sweep_ctr = sweep0 + (uint32_t)a.n_sweeps;
            if (s.bits_row) *s.bits_row = row0 + a.n_sweeps;
            atomicExch(s.arrive, 0u);
        }
    }
}

// LDS of a chain and the launch shape.  FP32 chains run here up to L = 8 (64 KB of
// a CU's 160 KB), FP64 ones up to L = 6: a chain has one CU, whose vector units the
// 2048 links of L = 8 keep busy three times as long as in FP32, while class passes
// spread few chains over all CUs (us per sweep here / class passes, L = 8 FP64 with
// replica exchange: 3 chains 243 / 127, 128 chains 257 / 198, 256 chains 264 / 271,
// 512 chains 511 / 432; L = 6 FP64: 3 chains 116 / 126, 256 chains 120 / 252; L = 8
// FP32: 3 chains 85 / 86, 256 chains 91 / 150).  Threads per block: with
// more chains than the 256 CUs an FP32 chain of L = 8 runs on 512 threads with
// 4 links each, so that two blocks share a CU and one computes while the other
// waits at a barrier; otherwise a chain gets up to 1024 threads, the shortest
// chain of dependent work per pass.  Measured, us per sweep of L = 8 FP32 with
// 1024 / 512 threads: 32 chains 70.3 / 78.7, 256 chains 71.2 / 80.0, 300
// chains 140.5 / 121.3, 512 chains 141.1 / 123.2.  The 512-thread shape's four links
// outgrow its 128 registers (16 spilled to 60 bytes of scratch per lane, 47 to 224 with
// the fused overrelaxation), and so do the link mode's shapes (10 to 30, 28 to 112
// bytes); the others have 0 to 20 bytes.  All chains of a context run in one launch,
// so one lattice that does not fit leaves every lattice to the class passes.
constexpr size_t kChainLds = 131072;
constexpr uint32_t kChainLinksF64 = 1024;
// Four lanes per link while the 4 x 128 links of L = 4 leave a CU's SIMDs two
// wavefronts each and every chain has a CU of its own; beyond that the work the
// lanes of a quad repeat (constants, new angle) costs more than the shorter chain
// of dependent instructions saves.  Measured, us per sweep one lane / four, L = 4:
// FP64 8 chains 49.2 / 42.8, 256 chains 48.4 / 43.1, 300 chains 70.9 / over 90;
// FP32 8 chains 20.4 / 18.7, 256 chains 20.5 / 19.0, 300 chains 24.8 / 29.
constexpr uint32_t kQuadLinks = 128;
constexpr int kQuadChains = 256;

static size_t chain_lds(uint32_t v2, size_t elem, bool per_link) {
    return v2 * (8 * elem + (per_link ? 8 + 3 * elem : 0));
}

// Whether every lattice's chain fits; per_link: with the candidates of a class
bool chain_fits(const LatTable& lt, size_t elem, bool per_link) {
    for (int i = 0; i < lt.n; ++i)
        if (chain_lds(lt.l[i].V2, elem, per_link) > kChainLds || (elem == 8 && lt.l[i].V2 > kChainLinksF64)) return false;
    return lt.n > 0;
}

template <typename T, int LPT, int MAXT, int VAR, int GRP = 1>
static hipError_t allow_lds() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_chain<T, LPT, MAXT, VAR, GRP>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)kChainLds);
}
template <typename T, int LPT, int MAXT>
static hipError_t shape_setup() {
    const hipError_t e = allow_lds<T, LPT, MAXT, kHbPlain>();
    return e == hipSuccess ? allow_lds<T, LPT, MAXT, kHbFuseOr>() : e;
}

// the current device's kernels may use more than the default 64 KB of LDS
hipError_t chain_setup() {
    hipError_t e = shape_setup<float, 1, 1024>();
    if (e == hipSuccess) e = shape_setup<float, 2, 1024>();
    if (e == hipSuccess) e = shape_setup<float, 4, 512>();
    if (e == hipSuccess) e = shape_setup<double, 1, 1024>();
    if (e == hipSuccess) e = allow_lds<float, 1, 1024, kHbPre>();
    if (e == hipSuccess) e = allow_lds<float, 2, 1024, kHbPre>();
    if (e == hipSuccess) e = allow_lds<double, 1, 1024, kHbPre>();
    return e;
}

template <typename T, int LPT, int MAXT, int VAR, int GRP = 1>
static void launch_var(const LatTable& lt, T* th, DevState s, const ChainArgs& a, uint32_t v2, hipStream_t st) {
    const dim3 gr(lt.n_chains), bl(((v2 + LPT - 1) / LPT * GRP + 63) / 64 * 64);
    hipLaunchKernelGGL((k_chain<T, LPT, MAXT, VAR, GRP>), gr, bl, chain_lds(v2, sizeof(T), VAR == kHbPre), st, lt, th, s, a);
}
template <typename T, int LPT, int MAXT, int GRP = 1>
static void launch_shape(const LatTable& lt, T* th, DevState s, const ChainArgs& a, uint32_t v2, hipStream_t st) {
    if (a.order == 1) launch_var<T, LPT, MAXT, kHbFuseOr, GRP>(lt, th, s, a, v2, st);
    else launch_var<T, LPT, MAXT, kHbPlain, GRP>(lt, th, s, a, v2, st);
}

template <typename T>
void launch_chain(const LatTable& lt, T* th, DevState s, const ChainArgs& a, hipStream_t st) {
    uint32_t v2 = 0;
    for (int i = 0; i < lt.n; ++i) v2 = v2 > lt.l[i].V2 ? v2 : lt.l[i].V2;
    if (a.mode == kModeLink) {
        if (v2 <= 1024) launch_var<T, 1, 1024, kHbPre>(lt, th, s, a, v2, st);
        else if constexpr (sizeof(T) == 4) launch_var<T, 2, 1024, kHbPre>(lt, th, s, a, v2, st);
        return;
    }
    if (v2 <= kQuadLinks && lt.n_chains <= kQuadChains) {
        launch_shape<T, 1, 512, 4>(lt, th, s, a, v2, st);
        return;
    }
    if (v2 <= 1024) {
        launch_shape<T, 1, 1024>(lt, th, s, a, v2, st);
        return;
    }
    if constexpr (sizeof(T) == 4) {   // chain_fits: FP64 chains have at most 1024 links per class
        if (lt.n_chains > 256) launch_shape<T, 4, 512>(lt, th, s, a, v2, st);
        else launch_shape<T, 2, 1024>(lt, th, s, a, v2, st);
    }
}

template void launch_chain<float>(const LatTable&, float*, DevState, const ChainArgs&, hipStream_t);
template void launch_chain<double>(const LatTable&, double*, DevState, const ChainArgs&, hipStream_t);

}  // namespace llr
