// llr_sweep.hip -- gfx950 kernels of the energy-restricted LLR sweep for 4D
// compact U(1) (arXiv:1509.08391, Sec. 2.2 restricted measure, Sec. 3.1 model).
//
// Layout: per chain, 2 planes x 8 colours x V/2 angles; colour c = 2 mu + p
// holds theta_mu at the sites of parity p, indexed by the half index
// h = s >> 1 of the lexicographic site s.  Links of one colour share no
// plaquette, so a colour class is updated in one data-parallel pass.
//
// A heatbath pass writes every proposal to the non-current plane of its
// colour, reduces the class Delta E per chain in int64 fixed point
// (order-independent, deterministic; one fence-free 64-bit atomic per block)
// and the last block of each chain takes the FP64 interval decision: on accept it flips the chain's current-plane
// bit, on reject nothing is written back.  An overrelaxation pass maps
// theta -> -2 phi - theta in place; it leaves every local action unchanged,
// so it needs neither a reduction nor a decision.
#include <hip/hip_runtime.h>

#include "llr_internal.hpp"
#include "llr_link.hpp"
#include "llr_walk.hpp"

namespace llr {


// links whose loads are in flight while one link's staples are summed
constexpr int kHbAhead = 1, kOrAhead = 1;

__device__ __forceinline__ int find_lat_site(const LatTable& lt, int b) {
    int li = 0;
#pragma unroll 1
    while (li + 1 < lt.n && b >= lt.l[li + 1].eblock0) ++li;
    return li;
}

// coordinates of the site with half index h and parity p
__device__ __forceinline__ void decode_half(const LatDev& L, uint32_t h, int p, int x[4]) {
    const uint32_t r1 = L.hL == 1 ? h : fdiv(h, L.mhL);   // ceil(2^32 / 1) does not fit 32 bits
    const int x0h = (int)(h - r1 * (uint32_t)L.hL);
    const uint32_t r2 = fdiv(r1, L.mL);
    x[1] = (int)(r1 - r2 * (uint32_t)L.L);
    const uint32_t r3 = fdiv(r2, L.mL);
    x[2] = (int)(r2 - r3 * (uint32_t)L.L);
    x[3] = (int)r3;
    x[0] = 2 * x0h + ((p + x[1] + x[2] + x[3]) & 1);
}
// Column tiles of the class passes.  The half index is h = pos + P x3 with
// pos = x0h + hL (x1 + L x2) the position in the (x0h, x1, x2) slab and
// P = hL L^2 its size, and the class's sites at one position and
// consecutive x3 alternate between x0 = 2 x0h and 2 x0h + 1 (the parity of
// x1 + x2 + x3 flips).  A tile is kBlock positions by LPT consecutive x3:
// thread tid owns position pos = pt kBlock + tid and x3 = xg LPT + r,
// r = 0..LPT-1, so its links share x0h, x1, x2 and the offsets along
// x1, x2, while x3 and its offsets are uniform over the wavefront.
struct ColTile {
    uint32_t pos;   // position in the slab; a lane past the slab's end gets 0
    uint32_t pos0;  // the tile's first position, pt kBlock
    bool in_slab;   // the lane's position lies in the slab (pt kBlock + tid < P)
    int x0h, x1, x2;
    int x3_0;       // x3 of the thread's first link
};
template <int LPT>
__device__ __forceinline__ ColTile col_tile(const LatDev& L, int tile, int tid) {
    ColTile t;
    int pt;
    const int xg = udiv(tile, L.npt, L.m_npt, pt);
    t.pos0 = (uint32_t)pt * kBlock;
    const uint32_t pos = t.pos0 + (uint32_t)tid;
    t.in_slab = pos < L.P;
    // a lane past the slab computes (and discards) the links of position 0,
    // so that its coordinates, neighbour offsets and addresses stay in range
    t.pos = t.in_slab ? pos : 0u;
    t.x3_0 = xg * LPT;
    const uint32_t r1 = L.hL == 1 ? t.pos : fdiv(t.pos, L.mhL);
    t.x0h = (int)(t.pos - r1 * (uint32_t)L.hL);
    const uint32_t r2 = fdiv(r1, L.mL);
    t.x1 = (int)(r1 - r2 * (uint32_t)L.L);
    t.x2 = (int)r2;
    return t;
}

template <typename T>
__device__ __forceinline__ T* chain_base(const LatDev& L, T* th, int cl) {
    return th + L.base + (long long)cl * 16ll * (long long)L.V2;
}
template <typename T>
__device__ __forceinline__ T* plane_ptr(T* chain, uint64_t curw, int c, uint32_t V2) {
    return chain + (size_t)((((curw >> (8 * c)) & 1ull) * 8ull) + (uint64_t)c) * V2;
}

// Element i of a plane through a 32-bit byte offset: the plane base is uniform
// (scalar registers) and every plane is < 4 GiB, so the access compiles to a
// global load/store with a scalar base and one 32-bit vector offset instead
// of a 64-bit vector address per access.
template <typename T>
__device__ __forceinline__ T ld_plane(const T* plane, uint32_t i) {
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(plane) + i * (uint32_t)sizeof(T));
}
template <typename T>
__device__ __forceinline__ void st_plane(T* plane, uint32_t i, T v) {
    *reinterpret_cast<T*>(reinterpret_cast<char*>(plane) + i * (uint32_t)sizeof(T)) = v;
}

// Half-index offsets of the neighbours of site x along each direction:
// up[nu] = h(x + nu) - h(x), dn[nu] = h(x - nu) - h(x), periodic.  Sites
// (2j, 2j+1) along x0 share a half index, so the x0 offsets depend on x0's
// parity; along nu >= 1 a step is L^nu / 2 half indices.
__device__ __forceinline__ void neighbour_offsets(const LatDev& L, const int x[4], int up[4], int dn[4]) {
    const int odd = x[0] & 1;
    up[0] = odd ? (x[0] == L.L - 1 ? 1 - L.hL : 1) : 0;
    dn[0] = odd ? 0 : (x[0] == 0 ? L.hL - 1 : -1);
#pragma unroll
    for (int nu = 1; nu < 4; ++nu) {
        // selects between per-lattice constants (no per-link multiply)
        up[nu] = x[nu] == L.L - 1 ? -L.hwrap[nu] : L.hstr[nu];
        dn[nu] = x[nu] == 0 ? L.hwrap[nu] : -L.hstr[nu];
    }
}

// A chain's 2 x 8 planes as one buffer resource.  An access is then base + lane
// offset + uniform offset with the uniform part (plane, x3 and a step along x3)
// in one scalar register: the lane offsets are computed once per column, a load
// costs one scalar add, and an address outside the chain is not accessed.
template <typename T>
struct ChainBuf {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ ChainBuf(T* chain, uint32_t V2)
        : r(__builtin_amdgcn_make_buffer_rsrc((void*)chain, 0, (int)(16u * V2 * (uint32_t)sizeof(T)), 0x00027000)) {}
    __device__ __forceinline__ T load(uint32_t lane, uint32_t uni) const {
        if constexpr (sizeof(T) == 4) {
            return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, (int)lane, (int)uni, 0));
        } else {
            return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, (int)lane, (int)uni, 0));
        }
    }
    __device__ __forceinline__ void store(uint32_t lane, uint32_t uni, T v) const {
        if constexpr (sizeof(T) == 4) {
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), r, (int)lane, (int)uni, 0);
        } else {
            typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, (int)lane, (int)uni, 0);
        }
    }
};

// Byte offset in the chain of colour c's current plane (other: the non-current)
template <typename T>
__device__ __forceinline__ uint32_t plane_off(uint64_t curw, int c, uint32_t V2, int other = 0) {
    return ((uint32_t)(((curw >> (8 * c)) & 1ull) ^ (uint64_t)other) * 8u + (uint32_t)c) * V2 * (uint32_t)sizeof(T);
}

// Lane byte offsets of a thread's column within a slab (see col_tile): its own
// position and the steps along x0, x1, x2.  The links' x0 = 2 x0h + b alternates
// in parity along the column, so the x0 steps come in two versions, for the
// column's even and odd links; the steps along x3 and the link's own shift P x3
// are uniform.
struct ColNbr {
    uint32_t pos;
    int up0[2], dn0[2];
    int up1, dn1, up2, dn2;
};
__device__ __forceinline__ ColNbr col_nbr(const LatDev& L, const ColTile& t, int p, int esz) {
    ColNbr n;
    const int b0 = (p + t.x1 + t.x2 + t.x3_0) & 1;   // x0 = 2 x0h + b0 for the even links
    const int uo = (t.x0h == L.hL - 1 ? 1 - L.hL : 1) * esz;  // x0 odd: the partner site 2 x0h + 2 (periodic)
    const int de = (t.x0h == 0 ? L.hL - 1 : -1) * esz;        // x0 even: the partner site 2 x0h - 1 (periodic)
    n.pos = t.pos * (uint32_t)esz;
    n.up0[0] = b0 ? uo : 0;
    n.dn0[0] = b0 ? 0 : de;
    n.up0[1] = b0 ? 0 : uo;
    n.dn0[1] = b0 ? de : 0;
    n.up1 = (t.x1 == L.L - 1 ? -L.hwrap[1] : L.hstr[1]) * esz;
    n.dn1 = (t.x1 == 0 ? L.hwrap[1] : -L.hstr[1]) * esz;
    n.up2 = (t.x2 == L.L - 1 ? -L.hwrap[2] : L.hstr[2]) * esz;
    n.dn2 = (t.x2 == 0 ? L.hwrap[2] : -L.hstr[2]) * esz;
    return n;
}

// Local field of link (MU, x): staples of the 2 x 3 plaquettes containing it,
// each oriented so that theta_MU(x) enters with a plus sign:
//   forward  s_f = th_nu(x+mu) - th_mu(x+nu) - th_nu(x)
//   backward s_b = th_nu(x-nu) - th_nu(x+mu-nu) - th_mu(x-nu)
// C + i S = sum of e^{i s}.  The link sits at slab position pos (per lane) and
// x3 (uniform); K = x3 parity relative to the column's first link selects the
// x0 offsets.

// A point in program order that v passes through: empty, but instructions that
// make v stay before it and those that use v after it.  Between the links of a
// thread it keeps the compiler from running several links' arithmetic side by
// side, whose live values would cost wavefronts (FP64: 256 registers).
template <typename T>
__device__ __forceinline__ void pin(T& v) {
    asm volatile("" : "+v"(v));
}
__device__ __forceinline__ void pin_uniform(int& v) { asm volatile("" : "+s"(v)); }

// A link's angles: per direction NU the six of its two plaquettes, and its own.
template <typename T>
struct LinkLoads {
    T v[3][6];
    T own;
};

// Issue the 19 loads of link (MU, x).
template <typename T, int MU, int K>
__device__ __forceinline__ void load_link(const LatDev& L, const ChainBuf<T>& cb, uint64_t curw, int p, const ColNbr& nb,
                                          int x3, LinkLoads<T>& q) {
    constexpr int E = (int)sizeof(T);
    const int vu[4] = {nb.up0[K], nb.up1, nb.up2, 0};
    const int vd[4] = {nb.dn0[K], nb.dn1, nb.dn2, 0};
    const int sh = (int)L.P * x3 * E;   // the link's own x3, uniform
    const int su[4] = {sh, sh, sh, sh + (x3 == L.L - 1 ? -L.hwrap[3] : L.hstr[3]) * E};
    const int sd[4] = {0, 0, 0, (x3 == 0 ? L.hwrap[3] : -L.hstr[3]) * E};
    const int o = p ^ 1;
    const uint32_t mu_q = plane_off<T>(curw, 2 * MU + o, L.V2);
#pragma unroll
    for (int NU = 0; NU < 4; ++NU) {
        if (NU == MU) continue;
        const int j = NU - (NU > MU ? 1 : 0);
        const uint32_t nu_p = plane_off<T>(curw, 2 * NU + p, L.V2);
        const uint32_t nu_q = plane_off<T>(curw, 2 * NU + o, L.V2);
        q.v[j][0] = cb.load(nb.pos + vu[MU], nu_q + su[MU]);                        // th_nu(x+mu)
        q.v[j][1] = cb.load(nb.pos + vu[NU], mu_q + su[NU]);                        // th_mu(x+nu)
        q.v[j][2] = cb.load(nb.pos, nu_p + sh);                                     // th_nu(x)
        q.v[j][3] = cb.load(nb.pos + (vu[MU] + vd[NU]), nu_p + su[MU] + sd[NU]);    // th_nu(x+mu-nu)
        q.v[j][4] = cb.load(nb.pos + vd[NU], mu_q + sh + sd[NU]);                   // th_mu(x-nu)
        q.v[j][5] = cb.load(nb.pos + vd[NU], nu_q + sh + sd[NU]);                   // th_nu(x-nu)
    }
    q.own = cb.load(nb.pos, plane_off<T>(curw, 2 * MU + p, L.V2) + sh);
}

template <typename T>
__device__ __forceinline__ void staple_sums(const LinkLoads<T>& q, T& C, T& S) {
    using M = Math<T>;
#pragma unroll
    for (int j = 0; j < 3; ++j) {   // the directions other than mu, ascending
        const T sf = q.v[j][0] - q.v[j][1] - q.v[j][2];
        const T sb = q.v[j][5] - q.v[j][3] - q.v[j][4];
        T s1, c1, s2, c2;
        M::sincos_rad(sf, &s1, &c1);
        M::sincos_rad(sb, &s2, &c2);
        if (j == 0) {   // the first direction seeds the sums
            C = c1 + c2;
            S = s1 + s2;
        } else {
            C += c1 + c2;
            S += s1 + s2;
        }
    }
}

// Staples and old angle of the LPT links of the thread's column.  The 19 loads
// of a link are issued together, AHEAD links before their sums: left alone, the
// scheduler saves registers by spreading them among the sums, one or two in
// flight at a time (heatbath of L = 20 x 128, FP32: 133 us so, 92 with a link's
// loads together, 88 with the next link's ahead).  Overrelaxation of L = 12 x 64
// FP32: 8.7 -> 7.4 us; of L = 20 x 128 67 -> 64, 5.7 TB/s.  Links past the lattice's
// end (x3 >= L, uniform) load the last one's and are computed, not used: with 4 links
// per thread a sixth of the links at L = 10, an eighth at L = 14, a tenth at L = 18,
// which the tuner weighs against fewer links per thread.
template <typename T, int MU, int LPT, int AHEAD>
__device__ __forceinline__ void col_staples(const LatDev& L, const ChainBuf<T>& cb, uint64_t curw, int p,
                                            const ColTile& ct, const ColNbr& nb, T* C, T* S, T* t_old) {
    LinkLoads<T> q[AHEAD + 1];
    auto load = [&](int r) __attribute__((always_inline)) {
        int x3 = min(ct.x3_0 + r, L.L - 1);
        pin_uniform(x3);
        if (r & 1) load_link<T, MU, 1>(L, cb, curw, p, nb, x3, q[r % (AHEAD + 1)]);
        else load_link<T, MU, 0>(L, cb, curw, p, nb, x3, q[r % (AHEAD + 1)]);
    };
#pragma unroll
    for (int r = 0; r < AHEAD && r < LPT; ++r) load(r);
#pragma unroll
    for (int r = 0; r < LPT; ++r) {
        if (r + AHEAD < LPT) load(r + AHEAD);
        __builtin_amdgcn_sched_barrier(0);
        staple_sums(q[r % (AHEAD + 1)], C[r], S[r]);
        t_old[r] = q[r % (AHEAD + 1)].own;
        pin(C[r]);
        pin(S[r]);
        pin(t_old[r]);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Sum of the wavefronts' values of a block, in thread 0.
__device__ __forceinline__ long long block_sum_i64(long long v) {
    __shared__ long long part[kBlock / 64];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) part[wid] = v;
    __syncthreads();
    long long tot = 0;
    if (threadIdx.x == 0) {
#pragma unroll
        for (int i = 0; i < kBlock / 64; ++i) tot += part[i];
    }
    return tot;
}

// Per-chain reduction without fences: each block adds, in ONE 64-bit atomic,
// 2^51 (its arrival) plus its partial sum in the lattice's fixed point 2^-fxb
// (two's complement in the low 51 bits; fxb is chosen so that 6V 2^fxb <=
// 2^49 bounds every partial sum).  The block whose addition brings the count
// to nblocks (< 2^13) holds the exact total, independent of arrival order.
__device__ __forceinline__ bool chain_arrive(unsigned long long* acc, long long part, int nblocks, long long* total) {
    const unsigned long long add = (1ull << 51) + (unsigned long long)part;
    const unsigned long long nw = atomicAdd(acc, add) + add;
    const long long S = ((long long)(nw << 13)) >> 13;
    const unsigned long long nb = (nw - (unsigned long long)S) >> 51;
    *total = S;
    return nb == (unsigned long long)nblocks;
}

// ---------------------------------------------------------------------------
// Heatbath class pass.  Link conditional ~ exp(a R cos(theta + phi)) with
// (C, S) the staple sums, R = |C + iS|, phi = arg(C + iS); theta' = X - phi
// with X ~ von Mises(a R) by Best & Fisher's wrapped-Cauchy envelope in its
// half-angle form: tan(X/2) = q tan(pi V1 / 2), q = (1 - rho)/(1 + rho).
// theta' is formed as arg[(cos(pi V1/2) + i q sin(pi V1/2))^2 (C - i S)], and
// the new local action is R cos X.
//
// Each thread owns the LPT class links of its column in a tile (a link's loads
// are issued one link ahead of its staple sums).  Sampler schedule: every link
// tries attempts 0 and 1 (one Philox call); the few links that reject both
// are queued in LDS and later rounds give each queued link its next two
// attempts with full lanes, so the lockstep cost of the acceptance tail is
// paid per block, not per wavefront.  Each link still takes its first
// accepted attempt in order.
// ---------------------------------------------------------------------------
template <typename T, int MU, int LPT, int VAR>
__device__ __forceinline__ void hb_block(const LatTable& lt, T* __restrict__ th, const DevState& s, int parity,
                                         int mode, int kind, uint32_t k0, uint32_t k1, int b) {
    using M = Math<T>;
    constexpr int NT = kBlock * LPT;
    // queued links keep only their |kappa|: the queue recomputes the sampler
    // constants (the same operations, so the same values), which keeps the
    // block's LDS small enough for one more resident block per CU
    __shared__ T s_ak[NT], s_ch[NT], s_sh[NT];
    __shared__ short s_queue[2][NT];
    __shared__ int s_qn[2];
    int li = 0;
#pragma unroll 1
    while (li + 1 < lt.n && b >= lt.l[li + 1].hb_block0) ++li;
    const LatDev& L = lt.l[li];
    if (mode == kModeApproach && s.lat_done[li]) return;
    const int rel = b - L.hb_block0;
    int tile;
    const int cl = udiv(rel, L.hb_bpc, L.m_hb, tile);
    const int g = L.chain0 + cl;
    const int colour = 2 * MU + parity;
    const int tid = threadIdx.x;
    const uint64_t curw = *reinterpret_cast<const uint64_t*>(s.cur + 8 * g);
    T* chain = chain_base(L, th, cl);
    const int gi = s.itv[g];
    const double acoup = mode == kModeApproach ? s.b[8 * g + colour] : (mode == kModeMuca ? s.mu_b[li] : s.a[gi]);
    const uint32_t sweep = kind == kApproach ? *s.approach_ctr : *s.sweep_ctr;
    const uint32_t c1base = ctr1_word(0, (uint32_t)colour, (uint32_t)kind, (uint32_t)L.lat_id);
    const uint32_t c3 = (uint32_t)(gi - L.itv0);
    const ChainBuf<T> cb(chain, L.V2);
    const uint32_t o_cur = plane_off<T>(curw, colour, L.V2);
    const uint32_t o_alt = plane_off<T>(curw, colour, L.V2, 1);
    // the fused pass's in-place store; a tuner's timing launch leaves the
    // state as it is and writes both angles into the non-current plane
    const uint32_t o_inpl = mode == kModeTune ? o_alt : o_cur;
    const ColTile ct = col_tile<LPT>(L, tile, tid);
    const ColNbr nb = col_nbr(L, ct, parity, (int)sizeof(T));
    const uint32_t pos = ct.pos;

    // Straight-line code per link: lanes past the slab compute position 0's
    // links and are masked where it matters (queue, stores, sums), and cases that
    // almost never occur branch on the whole wavefront.  Divergent branches here
    // cost a register copy per live value at every merge.
    T C[LPT], S[LPT], t_old[LPT], eps_old[LPT], R[LPT], ch[LPT], sh[LPT];
    T t_or_old[LPT];   // fused pass: the old angle's overrelaxation, from the sine and cosine at hand
    if (tid == 0) s_qn[0] = 0;
    col_staples<T, MU, LPT, kHbAhead>(L, cb, curw, parity, ct, nb, C, S, t_old);
#pragma unroll
    for (int r = 0; r < LPT; ++r) {
        T so, co;
        pin(C[r]);
        pin(S[r]);
        pin(t_old[r]);
        M::sincos_rad(t_old[r], &so, &co);
        eps_old[r] = fms2(C[r], co, S[r], so);
        if constexpr (VAR == kHbFuseOr) t_or_old[r] = or_angle_sc(t_old[r], so, co, C[r], S[r]);
        R[r] = M::sqrt_(fma2(C[r], C[r], S[r], S[r]));
        const T ak = M::abs_((T)acoup * R[r]);
        T q, rm1, kg2;
        vm_constants(ak, q, rm1, kg2);
        const uint4 w = philox10(make_uint4(pos + L.P * (uint32_t)(ct.x3_0 + r), c1base, sweep, c3), k0, k1);
        const bool ok = vm_first_two(w, ak, q, rm1, kg2, ch[r], sh[r]);
        ch[r] = ok ? ch[r] : T(2);   // no cosine: not accepted yet
        if constexpr (VAR == kHbFuseOr) pin(t_or_old[r]);
        pin(eps_old[r]);
        pin(R[r]);
        pin(ch[r]);
        pin(sh[r]);
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < LPT; ++r)
        if (ch[r] == T(2) && ct.in_slab && ct.x3_0 + r < L.L) {   // a link of the lattice
            const int e = r * kBlock + tid;
            s_queue[0][atomicAdd(&s_qn[0], 1)] = (short)e;
            s_ak[e] = M::abs_((T)acoup * R[r]);
            s_ch[e] = T(2);
        }
    __syncthreads();
    int cq = 0;
    // rounds after the first find a handful of links (0.7 % of the class): they
    // are dealt 2^lg lanes each, one attempt pair per lane, the first success in
    // attempt order wins, and the block is done
    for (int m = 1; m < kVmCap / 2;) {
        const int n = s_qn[cq];
        if (n == 0) break;
        if (tid == 0) s_qn[cq ^ 1] = 0;
        __syncthreads();
        int lg = 0;
        if (m > 1)
            while (lg < 4 && (n << (lg + 1)) <= 64 && m + (1 << (lg + 1)) <= kVmCap / 2) ++lg;
        const int sub = tid & ((1 << lg) - 1);
        for (int i = tid >> lg; i < n; i += kBlock >> lg) {
            const int e = s_queue[cq][i];
            // queue entry e = r kBlock + tid: link r of thread tid
            const uint32_t he = ct.pos0 + (uint32_t)(e & (kBlock - 1)) + L.P * (uint32_t)(ct.x3_0 + e / kBlock);
            const uint4 w = philox10(make_uint4(he, c1base | (uint32_t)(m + sub), sweep, c3), k0, k1);
            T qe, rme, kge;
            vm_constants(s_ak[e], qe, rme, kge);
            T che = T(1), she = T(0);
            const bool a0 = vm_attempt(w.x, w.y, qe, rme, kge, che, she);
            T c1, s1;
            const bool a1 = vm_try(w.z, w.w, qe, rme, kge, c1, s1);
            che = a0 ? che : c1;
            she = a0 ? she : s1;
            const unsigned long long ok = __ballot(a0 | a1);
            const int g0 = (tid & 63) & ~((1 << lg) - 1);   // the link's first lane
            const unsigned gm = (unsigned)(ok >> g0) & ((1u << (1 << lg)) - 1u);
            if (gm ? sub == __ffs((int)gm) - 1 : false) {
                s_ch[e] = che;
                s_sh[e] = she;
            }
            if (!gm && sub == 0) s_queue[cq ^ 1][atomicAdd(&s_qn[cq ^ 1], 1)] = (short)e;
        }
        __syncthreads();
        m += 1 << lg;
        cq ^= 1;
    }
    long long fx = 0;
    int fx32 = 0;   // FP32: the thread's class links at 2^-25 (|dE| <= 12 per link, LPT <= 4)
    if (ct.in_slab) {
#pragma unroll
        for (int r = 0; r < LPT; ++r) {
            const int x3 = ct.x3_0 + r;
            if (x3 >= L.L) continue;   // uniform
            const int e = r * kBlock + tid;
            if (ch[r] == T(2)) {
                ch[r] = s_ch[e];
                sh[r] = s_sh[e];
            }
            // a link at the attempt cap keeps its angle
            const bool lost = ch[r] == T(2);
            const uint32_t uni = L.P * (uint32_t)x3 * (uint32_t)sizeof(T);
            const T kap = (T)acoup * R[r];
            T dE, t_new, t_or_new;
            if constexpr (VAR == kHbFuseOr) hb_or_new_angle(ch[r], sh[r], C[r], S[r], R[r], kap, eps_old[r], t_or_new, dE);
            else hb_new_angle(ch[r], sh[r], C[r], S[r], R[r], kap, eps_old[r], t_new, dE);
            if (any_lane(lost)) {
                dE = lost ? T(0) : dE;
                if constexpr (VAR == kHbFuseOr) t_or_new = lost ? t_or_old[r] : t_or_new;
                else t_new = lost ? cb.load(nb.pos, o_cur + uni) : t_new;
            }
            if constexpr (VAR == kHbFuseOr) {
                // the class's overrelaxation follows at once, on the same staples:
                // of the heatbath candidate into the alternate plane, of the old
                // angle in place; the pass's decision picks the plane
                cb.store(nb.pos, o_alt + uni, t_or_new);
                cb.store(nb.pos, o_inpl + uni, t_or_old[r]);
            } else {
                cb.store(nb.pos, o_alt + uni, t_new);
            }
            if constexpr (VAR == kHbPre) {
                const size_t j = (size_t)L.lbase + (size_t)cl * L.V2 + L.P * (uint32_t)x3 + pos;
                T* lc = static_cast<T*>(s.link_cst);
                s.link_d[j] = lost ? kLinkNone : link_fixed(dE, L);
                lc[j] = C[r];
                lc[s.link_n + j] = S[r];
                lc[2 * s.link_n + j] = cb.load(nb.pos, o_cur + uni);
            }
            if constexpr (M::f32) fx32 += __float2int_rn(dE * 33554432.0f);
            else fx += to_fixed((double)dE, L);
        }
    }
    if constexpr (VAR == kHbPre) return;
    long long tot;
    if constexpr (M::f32) tot = block_sum_i64(wave_sum_i32(fx32)) << (L.fxb - 25);
    else tot = block_sum_i64(wave_sum_i64(fx));
    long long total = 0;
    if (threadIdx.x == 0 && chain_arrive(s.acc + (size_t)kAccStride * g, tot, L.hb_bpc, &total)) {
        const double E0 = s.E[g];
        const double En = E0 + (double)total * L.fxinv;
        const double lo = s.lo[gi], hi = s.hi[gi];
        bool acc;
        if (mode == kModeRestricted) {
            acc = En >= lo && En <= hi;
        } else if (mode == kModeApproach) {
            const double d0 = fmax(0.0, fmax(lo - E0, E0 - hi));
            const double d1 = fmax(0.0, fmax(lo - En, En - hi));
            acc = d1 <= d0;
            const double cen = s.cen[gi];
            const int sg = cen > En ? 1 : (cen < En ? -1 : 0);
            const int qq = 8 * g + colour;   // one coupling per colour class
            double eta = s.eta[qq];
            const int sp = s.sprev[qq];
            if (sp != 0 && sg != 0) eta = sg == sp ? fmin(0.05, 1.2 * eta) : fmax(1e-6, 0.5 * eta);
            s.eta[qq] = eta;
            s.b[qq] = fmin(4.0, fmax(0.0, s.b[qq] + eta * (double)sg));
            s.sprev[qq] = sg;
        } else if (mode == kModeMuca) {
            // target W(E) = 1/rho~(E), proposal the class heatbath at coupling
            // b: the proposal's normalisation depends only on the other
            // classes, so the Metropolis-Hastings ratio is
            // W(E')/W(E) e^{-b (E' - E)}
            const double lr = muca_lnw(L, s, En) - muca_lnw(L, s, E0) - acoup * (En - E0);
            const uint4 w = philox10(make_uint4(c3, ctr1_word(0, (uint32_t)colour, kMuca, (uint32_t)L.lat_id), sweep, 0u),
                                     k0, k1);
            acc = lr >= 0.0 || ((double)w.x + 0.5) * 0x1p-32 < exp(lr);
        } else {
            acc = mode == kModeFree;
        }
        if (mode != kModeTune) s.hb_prop[g] += 1ull;
        if (acc) {
            s.cur[8 * g + colour] ^= (uint8_t)1;
            s.E[g] = En;
            s.bits[g] |= (uint16_t)(1u << colour);
            s.hb_acc[g] += 1ull;
            if constexpr (VAR == kHbFuseOr) {
                if (mode != kModeTune) s.fu_acc[g] += 1ull;
            }
        }
        atomicExch(s.acc + (size_t)kAccStride * g, 0ull);
    }
}

// With 4 class links per thread the registers are kept to 72 (FP32, seven
// wavefronts per SIMD) and 128 (FP64, four).  They fit without scratch memory but
// for the fused FP64 pass, which spills two registers (12 bytes per lane); scalar
// registers beyond the limit (24 to 102) are kept in lanes of vector ones.
// The FP32 pass is bound by vector-instruction issue: 305 per class link (340
// before the straight-line links and the buffer addressing), of which about 45
// are a wavefront's prologue, queue and reduction shared by its 4 links.
// Heatbath of L = 20 x 128 FP32: 97.2 -> 88.4 us (six wavefronts 92, eight 89.6,
// a link's loads without the next link's ahead of it 91.9); L = 12 x 64 FP32, 2
// links: 16.1 -> 13.9 us; L = 12 x 64 FP64: 41.7 -> 39.4; the fused pass of
// L = 14 x 74: 26.7 -> 23.5.
template <typename T, int LPT, int VAR>
struct HbWaves { static constexpr int value = LPT == 4 ? (sizeof(T) == 4 ? 7 : 4) : 1; };

template <typename T, int MU, int LPT, int VAR>
__global__ __launch_bounds__(kBlock, (HbWaves<T, LPT, VAR>::value)) void k_hb(LatTable lt, T* __restrict__ th, DevState s, int parity, int mode,
                                               int kind, uint32_t k0, uint32_t k1, int reverse) {
    const int b0 = xcd_remap((int)blockIdx.x, (int)gridDim.x);
    hb_block<T, MU, LPT, VAR>(lt, th, s, parity, mode, kind, k0, k1, reverse ? (int)gridDim.x - 1 - b0 : b0);
}

constexpr int kWalkTile = 2048;          // class links of the per-link walk staged in LDS per tile

// Stage tile k of a chain's candidates (Delta E, staples, old angle) into LDS
// buffer `buf`, by threads [first, first + count) of the block; every thread
// issues its loads for several entries before its LDS stores, so a tile costs
// a few memory round trips, not one per entry.
template <typename T>
__device__ __forceinline__ void walk_stage(const DevState& s, size_t jb, uint32_t V2, int k, long long* sd, T* sc,
                                           T* ss, T* st, int first, int count) {
    constexpr int U = 8;
    const uint32_t t0 = (uint32_t)k * kWalkTile;
    const int nt = (int)min((uint32_t)kWalkTile, V2 - t0);
    const T* lc = static_cast<const T*>(s.link_cst);
    for (int base = (int)threadIdx.x - first; base < nt; base += U * count) {
        long long dd[U];
        T cc[U], sn[U], tt[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = base + u * count;
            if (i < nt) {
                const size_t j = jb + t0 + i;
                dd[u] = s.link_d[j];
                cc[u] = lc[j];
                sn[u] = lc[s.link_n + j];
                tt[u] = lc[2 * s.link_n + j];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = base + u * count;
            if (i < nt) {
                sd[i] = dd[u];
                sc[i] = cc[u];
                ss[i] = sn[u];
                st[i] = tt[u];
            }
        }
    }
}

// One block per chain.  The candidate pre-pass (k_hb<..., kHbPre>, mode
// kModeLinkPre) has written the candidates to the alternate plane and to the link
// buffers; the walk runs on wavefront 0 alone, with no barriers inside a tile,
// while wavefronts 1-3 stage the next tile into the other LDS buffer.
template <typename T, int MU>
__global__ __launch_bounds__(kBlock) void k_link_walk(LatTable lt, T* __restrict__ th, DevState s, int parity, int kind,
                                                      uint32_t k0, uint32_t k1) {
    __shared__ long long s_d[2][kWalkTile];
    __shared__ T s_c[2][kWalkTile], s_s[2][kWalkTile], s_t[2][kWalkTile];
    const int g = (int)blockIdx.x;
    int li = 0;
#pragma unroll 1
    while (li + 1 < lt.n && g >= lt.l[li + 1].chain0) ++li;
    const LatDev& L = lt.l[li];
    const int cl = g - L.chain0;
    const int colour = 2 * MU + parity;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const size_t jb = (size_t)L.lbase + (size_t)cl * L.V2;
    const int ntiles = (int)((L.V2 + kWalkTile - 1) / kWalkTile);
    walk_stage<T>(s, jb, L.V2, 0, s_d[0], s_c[0], s_s[0], s_t[0], 0, kBlock);
    __syncthreads();
    if (wid == 0) {
        const uint64_t curw = *reinterpret_cast<const uint64_t*>(s.cur + 8 * g);
        T* chain = chain_base(L, th, cl);
        const int own = (int)((curw >> (8 * colour)) & 1ull);
        T* palt = chain + (size_t)((own ^ 1) * 8 + colour) * L.V2;
        const int gi = s.itv[g];
        const double E0 = s.E[g];
        Walk w = walk_begin(L, colour, kind, *s.sweep_ctr, (uint32_t)(gi - L.itv0), k0, k1, s.a[gi], E0, s.lo[gi],
                            s.hi[gi]);
        for (int k = 0; k < ntiles; ++k) {
            const int buf = k & 1;
            const uint32_t t0 = (uint32_t)k * kWalkTile;
            const int nt = (int)min((uint32_t)kWalkTile, L.V2 - t0);
            walk_links<T>(L, w, t0, nt, s_d[buf], s_c[buf], s_s[buf], s_t[buf],
                          [&](uint32_t h, T v) { st_plane(palt, h, v); });
            __syncthreads();   // pairs with the stagers' barrier of this tile
        }
        if (lane == 0) {
            s.E[g] = E0 + (double)w.Ssum * w.fxwinv;
            s.cur[8 * g + colour] ^= (uint8_t)1;
            s.bits[g] |= (uint16_t)(1u << colour);
            s.hb_prop[g] += 1ull;
            s.hb_acc[g] += 1ull;
            s.link_fix[g] += w.fixes;
            s.link_arc[g] += w.arcs;
        }
    } else {
        for (int k = 0; k < ntiles; ++k) {
            if (k + 1 < ntiles) {
                const int nb = (k + 1) & 1;
                walk_stage<T>(s, jb, L.V2, k + 1, s_d[nb], s_c[nb], s_s[nb], s_t[nb], 64, kBlock - 64);
            }
            __syncthreads();   // tile k walked, tile k + 1 staged
        }
    }
}

// ---------------------------------------------------------------------------
// Overrelaxation class pass: theta' = arg[(C - i S)^2 e^{-i theta}] = -2 phi - theta,
// LPT class links per thread.
// ---------------------------------------------------------------------------
template <typename T, int MU, int LPT>
__device__ __forceinline__ void or_block(const LatTable& lt, T* __restrict__ th, const DevState& s, int parity,
                                         int to_alt, int b) {
    using M = Math<T>;
    constexpr int NT = kBlock * LPT;
    int li = 0;
#pragma unroll 1
    while (li + 1 < lt.n && b >= lt.l[li + 1].or_block0) ++li;
    const LatDev& L = lt.l[li];
    const int rel = b - L.or_block0;
    int tile;
    const int cl = udiv(rel, L.or_bpc, L.m_or, tile);
    const int g = L.chain0 + cl;
    const int colour = 2 * MU + parity;
    const uint64_t curw = *reinterpret_cast<const uint64_t*>(s.cur + 8 * g);
    T* chain = chain_base(L, th, cl);
    const ChainBuf<T> cb(chain, L.V2);
    // timing runs of the tuner write to the non-current plane (state unchanged)
    const uint32_t o_out = plane_off<T>(curw, colour, L.V2, to_alt ? 1 : 0);
    const ColTile ct = col_tile<LPT>(L, tile, (int)threadIdx.x);
    const ColNbr nb = col_nbr(L, ct, parity, (int)sizeof(T));
    T C[LPT], S[LPT], t_old[LPT];
    col_staples<T, MU, LPT, kOrAhead>(L, cb, curw, parity, ct, nb, C, S, t_old);
#pragma unroll
    for (int r = 0; r < LPT; ++r) {
        const int x3 = ct.x3_0 + r;
        if (x3 >= L.L) continue;   // uniform
        const T t_new = or_angle(t_old[r], C[r], S[r]);
        if (ct.in_slab) cb.store(nb.pos, o_out + L.P * (uint32_t)x3 * (uint32_t)sizeof(T), t_new);
    }
}

template <typename T, int MU, int LPT>
__global__ __launch_bounds__(kBlock) void k_or(LatTable lt, T* __restrict__ th, DevState s, int parity, int to_alt,
                                               int reverse) {
    const int b0 = xcd_remap((int)blockIdx.x, (int)gridDim.x);
    or_block<T, MU, LPT>(lt, th, s, parity, to_alt, reverse ? (int)gridDim.x - 1 - b0 : b0);
}


// ---------------------------------------------------------------------------
// Full FP64 energy: E = sum_{x, mu<nu} cos theta_{mu nu}(x), one thread per
// site.  The first half of a chain's blocks takes the even sites, the second
// half the odd ones, so the parity and with it every plane base is uniform
// over a block.  check (kCheck* bits) adds the health tests of the chain's
// incremental E before it is replaced: any non-finite plaquette angle, the
// drift against the recomputed E, and the recomputed E against the chain's
// restriction; failures set sticky kHealth* flags that the host reads.
// ---------------------------------------------------------------------------
template <typename T, bool OBS>
__global__ __launch_bounds__(kBlock) void k_energy(LatTable lt, const T* __restrict__ th, DevState s, int check) {
    const int b = xcd_remap((int)blockIdx.x, (int)gridDim.x);
    const int li = find_lat_site(lt, b);
    const LatDev& L = lt.l[li];
    const int rel = b - L.eblock0;
    const int cl = rel / L.ebpc;
    const int tile = rel - cl * L.ebpc;
    const int g = L.chain0 + cl;
    const uint64_t curw = *reinterpret_cast<const uint64_t*>(s.cur + 8 * g);
    const T* chain = chain_base(L, const_cast<T*>(th), cl);
    const int half = L.ebpc >> 1;
    const int p = tile >= half ? 1 : 0;
    const uint32_t h = (uint32_t)(tile - p * half) * kBlock + threadIdx.x;
    long long fx = 0, fa = 0;
    int bad = 0;   // a plaquette angle that is not finite
    if (h < L.V2) {
        int x[4];
        decode_half(L, h, p, x);
        double own[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) own[m] = (double)ld_plane(plane_ptr(chain, curw, 2 * m + p, L.V2), h);
        int upo[4], dno[4];
        neighbour_offsets(L, x, upo, dno);
        uint32_t hup[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) hup[m] = h + upo[m];
#pragma unroll
        for (int mu = 0; mu < 4; ++mu)
#pragma unroll
            for (int nu = mu + 1; nu < 4; ++nu) {
                const double t_nu_pmu = (double)ld_plane(plane_ptr(chain, curw, 2 * nu + (p ^ 1), L.V2), hup[mu]);
                const double t_mu_pnu = (double)ld_plane(plane_ptr(chain, curw, 2 * mu + (p ^ 1), L.V2), hup[nu]);
                const double ang = own[mu] + t_nu_pmu - t_mu_pnu - own[nu];
                bad |= !(fabs(ang) < INFINITY);
                const double cp = cos_plaq(ang);
                fx += __double2ll_rn(cp * L.fx);
                if (OBS) fa += __double2ll_rn(__fma_rn(2.0 * cp, cp, -1.0) * L.fx);   // cos 2 theta_P
            }
    }
    if (__syncthreads_or(bad) && threadIdx.x == 0) atomicOr(s.health + g, (uint32_t)kHealthNonFinite);
    const long long tot = block_sum_i64(wave_sum_i64(fx));
    long long total = 0;
    if (threadIdx.x == 0 && chain_arrive(s.eacc + (size_t)kAccStride * g, tot, L.ebpc, &total)) {
        const double En = (double)total * L.fxinv;
        if (check) {
            // health of the chain's incremental E: its drift from the
            // recomputed value, and (restricted sweeps) that the recomputed E
            // lies in the chain's restriction up to that drift bound
            const double bound = (sizeof(T) == 4 ? 1e-5 : 1e-9) * 12.0 * (double)L.V2;
            const double d = fabs(En - s.E[g]);
            uint32_t f = 0;
            if (check & kCheckDrift) {
                s.drift[g] = fmax(s.drift[g], d);
                if (!(d <= bound)) f |= kHealthDrift;
            }
            if (check & kCheckInterval) {
                const int gi = s.itv[g];
                if (!(En >= s.lo[gi] - bound && En <= s.hi[gi] + bound)) f |= kHealthOutside;
            }
            if (f) atomicOr(s.health + g, f);
        }
        s.E[g] = En;
        atomicExch(s.eacc + (size_t)kAccStride * g, 0ull);
    }
    if (OBS) {
        __syncthreads();   // block_sum_i64's shared partials are reused
        const long long ta = block_sum_i64(wave_sum_i64(fa));
        long long tb = 0;
        if (threadIdx.x == 0 && chain_arrive(s.oacc + (size_t)kAccStride * g, ta, L.ebpc, &tb)) {
            s.obs[g] = (double)tb * L.fxinv;
            atomicExch(s.oacc + (size_t)kAccStride * g, 0ull);
        }
    }
}

// ---------------------------------------------------------------------------
// Hot start: theta = -pi + 2 pi U (kind 1, w0 = mu V + s, w3 = chain index),
// computed in FP64 with one fused multiply-add and rounded to the precision.
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(kBlock) void k_hot_start(LatTable lt, T* __restrict__ th, DevState s, uint32_t k0,
                                                      uint32_t k1) {
    const int b = (int)blockIdx.x;
    const int li = find_lat_site(lt, b);
    const LatDev& L = lt.l[li];
    const int rel = b - L.eblock0;
    const int cl = rel / L.ebpc;
    const int tile = rel - cl * L.ebpc;
    const int g = L.chain0 + cl;
    T* chain = chain_base(L, th, cl);
    const uint32_t V = 2u * L.V2;
    const uint32_t sidx = (uint32_t)tile * kBlock + threadIdx.x;   // lexicographic site
    if (sidx < V) {
        const uint32_t r1 = fdiv(sidx, L.mL);
        const int x0 = (int)(sidx - r1 * (uint32_t)L.L);
        const uint32_t r2 = fdiv(r1, L.mL);
        const int x1 = (int)(r1 - r2 * (uint32_t)L.L);
        const uint32_t r3 = fdiv(r2, L.mL);
        const int x2 = (int)(r2 - r3 * (uint32_t)L.L);
        const int x3 = (int)r3;
        const int p = (x0 + x1 + x2 + x3) & 1;
        const uint32_t h = sidx >> 1;
        for (int mu = 0; mu < 4; ++mu) {
            const uint4 w = philox10(make_uint4((uint32_t)mu * V + sidx, ctr1_word(0, 0, kInit, (uint32_t)L.lat_id), 0u,
                                                (uint32_t)cl),
                                     k0, k1);
            const double u = Math<T>::f32 ? ((double)(w.x >> 9) + 0.5) * 0x1p-23 : ((double)w.x + 0.5) * 0x1p-32;
            const double t = __fma_rn(6.28318530717958647692, u, -3.14159265358979323846);
            chain[(size_t)(2 * mu + p) * L.V2 + h] = (T)t;
        }
    }
    if (threadIdx.x == 0 && tile == 0) {
        *reinterpret_cast<uint64_t*>(s.cur + 8 * g) = 0ull;
        s.itv[g] = g;
        s.conf[g] = g;
    }
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_export(LatDev L, const T* __restrict__ th, DevState s, T* __restrict__ out) {
    const long long V = 2ll * L.V2;
    const long long i = (long long)blockIdx.x * kBlock + threadIdx.x;   // over chains x 4 x V
    if (i >= (long long)L.n_chains * 4 * V) return;
    const int cl = (int)(i / (4 * V));
    const long long r = i - (long long)cl * 4 * V;
    const int mu = (int)(r / V);
    const uint32_t sidx = (uint32_t)(r - (long long)mu * V);
    const uint32_t r1 = fdiv(sidx, L.mL);
    const int x0 = (int)(sidx - r1 * (uint32_t)L.L);
    const uint32_t r2 = fdiv(r1, L.mL);
    const int x1 = (int)(r1 - r2 * (uint32_t)L.L);
    const uint32_t r3 = fdiv(r2, L.mL);
    const int x2 = (int)(r2 - r3 * (uint32_t)L.L);
    const int p = (x0 + x1 + x2 + (int)r3) & 1;
    const uint64_t curw = *reinterpret_cast<const uint64_t*>(s.cur + 8 * (L.chain0 + cl));
    const T* chain = chain_base(L, const_cast<T*>(th), cl);
    out[i] = plane_ptr(chain, curw, 2 * mu + p, L.V2)[sidx >> 1];
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_import(LatDev L, T* __restrict__ th, DevState s, const T* __restrict__ in) {
    const long long V = 2ll * L.V2;
    const long long i = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (i >= (long long)L.n_chains * 4 * V) return;
    const int cl = (int)(i / (4 * V));
    const long long r = i - (long long)cl * 4 * V;
    const int mu = (int)(r / V);
    const uint32_t sidx = (uint32_t)(r - (long long)mu * V);
    const uint32_t r1 = fdiv(sidx, L.mL);
    const int x0 = (int)(sidx - r1 * (uint32_t)L.L);
    const uint32_t r2 = fdiv(r1, L.mL);
    const int x1 = (int)(r1 - r2 * (uint32_t)L.L);
    const uint32_t r3 = fdiv(r2, L.mL);
    const int x2 = (int)(r2 - r3 * (uint32_t)L.L);
    const int p = (x0 + x1 + x2 + (int)r3) & 1;
    T* chain = chain_base(L, th, cl);
    chain[(size_t)(2 * mu + p) * L.V2 + (sidx >> 1)] = in[i];
    if (r == 0) {
        const int g = L.chain0 + cl;
        *reinterpret_cast<uint64_t*>(s.cur + 8 * g) = 0ull;
        s.itv[g] = g;
        s.conf[g] = g;
    }
}

__global__ __launch_bounds__(1024) void k_obs_row(int n, DevState s, double* __restrict__ E_row,
                                                  double* __restrict__ B_row) {
    for (int k = threadIdx.x; k < n; k += blockDim.x) {
        const int g = s.conf[k];
        E_row[k] = s.E[g];
        B_row[k] = s.obs[g];
    }
}

// ---------------------------------------------------------------------------
// End of a sweep, one block: replica exchange, the measured energy of every
// interval, the accept bits to the log, the sweep counter.  A chain of dependent
// loads on a few KB, 6.5 us of which most is the launch: one kernel for what two
// took 10 us for.
// ---------------------------------------------------------------------------
// Replica exchange (Sec. 2.5) between intervals k and k+1 of one lattice, for
// k = t (mod 2) at sweep t; eligible iff each configuration lies in the other
// interval; accepted with min(1, exp[(a_k - a_{k+1})(E_{k+1} - E_k)]).  Only
// the chain <-> interval labels move.
__device__ __forceinline__ void replica_pairs(const LatTable& lt, const DevState& s, uint32_t t, uint32_t k0, uint32_t k1) {
    unsigned long long prop = 0, accd = 0;
    for (int li = 0; li < lt.n; ++li) {
        const LatDev& L = lt.l[li];
        const int npair = (L.n_chains - (int)(t & 1u)) / 2;
        for (int i = threadIdx.x; i < npair; i += blockDim.x) {
            const int k = 2 * i + (int)(t & 1u);
            if (k + 1 >= L.n_chains) continue;
            const int kg = L.chain0 + k;
            const int A = s.conf[kg], B = s.conf[kg + 1];
            const double EA = s.E[A], EB = s.E[B];
            if (!(EA >= s.lo[kg + 1] && EA <= s.hi[kg + 1] && EB >= s.lo[kg] && EB <= s.hi[kg])) continue;
            const uint4 w = philox10(make_uint4((uint32_t)k, ctr1_word(0, 0, kReplica, (uint32_t)L.lat_id), t, 0u), k0, k1);
            const double u = ((double)w.x + 0.5) * 0x1p-32;
            const double xx = (s.a[kg] - s.a[kg + 1]) * (EB - EA);
            ++prop;
            if (xx >= 0.0 || u < exp(xx)) {
                s.conf[kg] = B;
                s.conf[kg + 1] = A;
                s.itv[A] = kg + 1;
                s.itv[B] = kg;
                ++accd;
            }
        }
    }
    if (prop) atomicAdd(s.re_cnt, prop);
    if (accd) atomicAdd(s.re_cnt + 1, accd);
}

// Overrelaxation passes are always accepted (E unchanged): their bits 8..15
// are set here for sweeps that ran them.
__global__ __launch_bounds__(1024) void k_end_sweep(LatTable lt, DevState s, int replica, int measure, int approach,
                                                    int with_or, uint32_t k0, uint32_t k1, double* __restrict__ E_row,
                                                    uint16_t* __restrict__ b_row) {
    const int n = lt.n_chains;
    const long long row = s.bits_row ? *s.bits_row : 0;
    const uint32_t t = approach ? *s.approach_ctr : *s.sweep_ctr;
    for (int g = threadIdx.x; g < n; g += blockDim.x) {
        const uint16_t bits = (uint16_t)(s.bits[g] | (with_or ? 0xff00u : 0u));
        if (s.bits_log && row < s.bits_rows_max) s.bits_log[row * n + g] = bits;
        s.bits_last[g] = bits;
        s.bits[g] = 0;
        if (E_row) E_row[g] = s.E[g];
        if (b_row) b_row[g] = bits;
    }
    if (replica) replica_pairs(lt, s, t, k0, k1);
    __syncthreads();   // every label is final, every thread has read the counters
    if (measure)
        for (int g = threadIdx.x; g < n; g += blockDim.x) s.sumE[s.itv[g]] += s.E[g];
    if (threadIdx.x == 0) {
        if (approach) *s.approach_ctr = t + 1u;
        else *s.sweep_ctr = t + 1u;
        if (s.bits_row) *s.bits_row = row + 1;
    }
}

// Robbins-Monro step of every interval (eq. (kk21), Algorithm 1 sign):
// a^(n+1) = a^(n) - 12 (mean - c_k) / ((n + 1) w^2).
__global__ __launch_bounds__(1024) void k_rm_update(int n, DevState s, RunCfg cfg) {
    const int it = *s.rm_iter;
    for (int k = threadIdx.x; k < n; k += blockDim.x) {
        const double mean = s.sumE[k] / (double)cfg.n_a;
        const double a0 = s.a[k];
        const double wk = s.w[k];
        const double an = a0 - 12.0 * (mean - s.cen[k]) / ((double)(it + 1) * wk * wk);
        const double da = an - a0;
        s.a[k] = an;
        s.a_hist[(long long)(it + 1) * n + k] = an;
        if (s.conv_iter[k] < 0 && fabs(da) < cfg.eps) {
            s.conv_iter[k] = it;
            s.conv_sweeps[k] = (long long)(it + 1) * cfg.nsw;   // approach sweeps added on the host
        }
        s.sumE[k] = 0.0;
    }
    __syncthreads();
    if (threadIdx.x == 0) *s.rm_iter = it + 1;
}

__global__ __launch_bounds__(1024) void k_approach_init(int n, DevState s) {
    for (int q = threadIdx.x; q < 8 * n; q += blockDim.x) {
        s.b[q] = s.a[s.itv[q >> 3]];
        s.eta[q] = 0.05;
        s.sprev[q] = 0;
    }
}

__global__ __launch_bounds__(1024) void k_approach_check(LatTable lt, DevState s) {
    __shared__ int outside[kMaxLat];
    if (threadIdx.x < kMaxLat) outside[threadIdx.x] = 0;
    __syncthreads();
    for (int li = 0; li < lt.n; ++li) {
        const LatDev& L = lt.l[li];
        for (int c = threadIdx.x; c < L.n_chains; c += blockDim.x) {
            const int g = L.chain0 + c;
            const int k = s.itv[g];
            const double E = s.E[g];
            if (!(E >= s.lo[k] && E <= s.hi[k])) atomicAdd(&outside[li], 1);
        }
    }
    __syncthreads();
    if (threadIdx.x < (unsigned)lt.n) s.lat_outside[threadIdx.x] = outside[threadIdx.x];
}

__global__ void k_test_philox(long n, const uint4* __restrict__ ctr, uint32_t k0, uint32_t k1, uint4* __restrict__ out) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = philox10(ctr[i], k0, k1);
}

// Stand-alone draws of the heatbath sampler (same arithmetic as k_hb, attempts
// taken sequentially).
template <typename T>
__global__ void k_test_vonmises(long n, double kappa, uint32_t k0, uint32_t k1, uint32_t c1, uint32_t c2, uint32_t c3,
                                double* X, int* att) {
    using M = Math<T>;
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const T ak = (T)kappa;
    T q, rm1, kg2;
    vm_constants(ak, q, rm1, kg2);
    int a = 0;
    T ch = T(1), sh = T(0);
    for (int m = 0; m < kVmCap / 2 && !a; ++m) {
        const uint4 w = philox10(make_uint4((uint32_t)i, c1 | (uint32_t)m, c2, c3), k0, k1);
        if (ak == T(0)) { M::sincos_halfpi_w(w.x, &sh, &ch); a = 1; break; }
        if (vm_attempt(w.x, w.y, q, rm1, kg2, ch, sh)) a = 2 * m + 1;
        else if (vm_attempt(w.z, w.w, q, rm1, kg2, ch, sh)) a = 2 * m + 2;
    }
    att[i] = a;
    X[i] = a ? 2.0 * (double)M::atan2_(sh, ch) : 0.0;
}

// ------------------------------------------------------------------ launchers
template <typename T>
void launch_hot_start(const LatTable& lt, T* th, DevState s, uint32_t k0, uint32_t k1, hipStream_t st) {
    hipLaunchKernelGGL(k_hot_start<T>, dim3(lt.site_blocks), dim3(kBlock), 0, st, lt, th, s, k0, k1);
}

// VAR: kHbPlain, the candidate pre-pass of the per-link constraint (kHbPre),
// or the pass followed by the class's overrelaxation (kHbFuseOr); separate
// instantiations, so that the plain pass carries none of the others' code
template <typename T, int LPT, int VAR>
static void hb_dispatch(const LatTable& lt, T* th, DevState s, int colour, int mode, int kind, uint32_t k0,
                        uint32_t k1, hipStream_t st) {
    const int p = colour & 1;
    const int rv = lt.serpentine ? p : 0;
    dim3 gr(lt.hb_blocks), bl(kBlock);
    switch (colour >> 1) {
        case 0: hipLaunchKernelGGL((k_hb<T, 0, LPT, VAR>), gr, bl, 0, st, lt, th, s, p, mode, kind, k0, k1, rv); break;
        case 1: hipLaunchKernelGGL((k_hb<T, 1, LPT, VAR>), gr, bl, 0, st, lt, th, s, p, mode, kind, k0, k1, rv); break;
        case 2: hipLaunchKernelGGL((k_hb<T, 2, LPT, VAR>), gr, bl, 0, st, lt, th, s, p, mode, kind, k0, k1, rv); break;
        default: hipLaunchKernelGGL((k_hb<T, 3, LPT, VAR>), gr, bl, 0, st, lt, th, s, p, mode, kind, k0, k1, rv); break;
    }
}

template <typename T, int VAR>
static void hb_tiles(const LatTable& lt, T* th, DevState s, int colour, int mode, int kind, uint32_t k0, uint32_t k1,
                     hipStream_t st) {
    switch (lt.hb_lpt) {
        case 1: hb_dispatch<T, 1, VAR>(lt, th, s, colour, mode, kind, k0, k1, st); break;
        case 2: hb_dispatch<T, 2, VAR>(lt, th, s, colour, mode, kind, k0, k1, st); break;
        default: hb_dispatch<T, 4, VAR>(lt, th, s, colour, mode, kind, k0, k1, st); break;
    }
}

template <typename T>
void launch_hb_pass(const LatTable& lt, T* th, DevState s, int colour, int mode, int kind, uint32_t k0, uint32_t k1,
                    hipStream_t st) {
    if (mode != kModeLink) {
        hb_tiles<T, kHbPlain>(lt, th, s, colour, mode, kind, k0, k1, st);
        return;
    }
    hb_tiles<T, kHbPre>(lt, th, s, colour, kModeLinkPre, kind, k0, k1, st);
    const int p = colour & 1;
    dim3 gr(lt.n_chains), bl(kBlock);
    switch (colour >> 1) {
        case 0: hipLaunchKernelGGL((k_link_walk<T, 0>), gr, bl, 0, st, lt, th, s, p, kind, k0, k1); break;
        case 1: hipLaunchKernelGGL((k_link_walk<T, 1>), gr, bl, 0, st, lt, th, s, p, kind, k0, k1); break;
        case 2: hipLaunchKernelGGL((k_link_walk<T, 2>), gr, bl, 0, st, lt, th, s, p, kind, k0, k1); break;
        default: hipLaunchKernelGGL((k_link_walk<T, 3>), gr, bl, 0, st, lt, th, s, p, kind, k0, k1); break;
    }
}

template <typename T>
void launch_hb_or_pass(const LatTable& lt, T* th, DevState s, int colour, int mode, uint32_t k0, uint32_t k1,
                       hipStream_t st) {
    hb_tiles<T, kHbFuseOr>(lt, th, s, colour, mode, kSweep, k0, k1, st);
}

template <typename T, int LPT>
static void or_dispatch(const LatTable& lt, T* th, DevState s, int colour, int to_alt, hipStream_t st) {
    const int p = colour & 1;
    const int rv = lt.serpentine ? p : 0;
    dim3 gr(lt.or_blocks), bl(kBlock);
    switch (colour >> 1) {
        case 0: hipLaunchKernelGGL((k_or<T, 0, LPT>), gr, bl, 0, st, lt, th, s, p, to_alt, rv); break;
        case 1: hipLaunchKernelGGL((k_or<T, 1, LPT>), gr, bl, 0, st, lt, th, s, p, to_alt, rv); break;
        case 2: hipLaunchKernelGGL((k_or<T, 2, LPT>), gr, bl, 0, st, lt, th, s, p, to_alt, rv); break;
        default: hipLaunchKernelGGL((k_or<T, 3, LPT>), gr, bl, 0, st, lt, th, s, p, to_alt, rv); break;
    }
}

template <typename T>
void launch_or_pass(const LatTable& lt, T* th, DevState s, int colour, int to_alt, hipStream_t st) {
    switch (lt.or_lpt) {
        case 1: or_dispatch<T, 1>(lt, th, s, colour, to_alt, st); break;
        case 2: or_dispatch<T, 2>(lt, th, s, colour, to_alt, st); break;
        default: or_dispatch<T, 4>(lt, th, s, colour, to_alt, st); break;
    }
}

template <typename T>
void launch_energy(const LatTable& lt, const T* th, DevState s, hipStream_t st, bool with_obs, int check) {
    if (with_obs) hipLaunchKernelGGL((k_energy<T, true>), dim3(lt.site_blocks), dim3(kBlock), 0, st, lt, th, s, check);
    else hipLaunchKernelGGL((k_energy<T, false>), dim3(lt.site_blocks), dim3(kBlock), 0, st, lt, th, s, check);
}

template <typename T>
void launch_export(const LatTable& lt, int li, const T* th, DevState s, T* out, hipStream_t st) {
    const LatDev& L = lt.l[li];
    const long long n = (long long)L.n_chains * 8ll * L.V2;
    hipLaunchKernelGGL(k_export<T>, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, L, th, s, out);
}

template <typename T>
void launch_import(const LatTable& lt, int li, T* th, DevState s, const T* in, hipStream_t st) {
    const LatDev& L = lt.l[li];
    const long long n = (long long)L.n_chains * 8ll * L.V2;
    hipLaunchKernelGGL(k_import<T>, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, L, th, s, in);
}

void launch_end_sweep(const LatTable& lt, DevState s, int replica, int measure, int approach, int with_or,
                      uint32_t k0, uint32_t k1, double* E_row, uint16_t* b_row, hipStream_t st) {
    hipLaunchKernelGGL(k_end_sweep, dim3(1), dim3(1024), 0, st, lt, s, replica, measure, approach, with_or, k0, k1, E_row,
                       b_row);
}
void launch_obs_row(const LatTable& lt, DevState s, double* E_row, double* B_row, hipStream_t st) {
    hipLaunchKernelGGL(k_obs_row, dim3(1), dim3(1024), 0, st, lt.n_chains, s, E_row, B_row);
}
void launch_rm_update(const LatTable& lt, DevState s, RunCfg cfg, hipStream_t st) {
    hipLaunchKernelGGL(k_rm_update, dim3(1), dim3(1024), 0, st, lt.n_chains, s, cfg);
}
void launch_approach_init(const LatTable& lt, DevState s, hipStream_t st) {
    hipLaunchKernelGGL(k_approach_init, dim3(1), dim3(1024), 0, st, lt.n_chains, s);
}
void launch_approach_check(const LatTable& lt, DevState s, hipStream_t st) {
    hipLaunchKernelGGL(k_approach_check, dim3(1), dim3(1024), 0, st, lt, s);
}
void launch_test_philox(long n, const uint4* ctr, uint32_t k0, uint32_t k1, uint4* out, hipStream_t st) {
    hipLaunchKernelGGL(k_test_philox, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, ctr, k0, k1, out);
}
template <typename T>
void launch_test_vonmises(long n, double kappa, uint32_t k0, uint32_t k1, uint32_t c1, uint32_t c2, uint32_t c3,
                          double* X, int* att, hipStream_t st) {
    hipLaunchKernelGGL(k_test_vonmises<T>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, kappa, k0, k1, c1,
                       c2, c3, X, att);
}

#define LLR_INST(T)                                                                                              \
    template void launch_hot_start<T>(const LatTable&, T*, DevState, uint32_t, uint32_t, hipStream_t);          \
    template void launch_hb_pass<T>(const LatTable&, T*, DevState, int, int, int, uint32_t, uint32_t, hipStream_t); \
    template void launch_or_pass<T>(const LatTable&, T*, DevState, int, int, hipStream_t);                           \
    template void launch_hb_or_pass<T>(const LatTable&, T*, DevState, int, int, uint32_t, uint32_t, hipStream_t);     \
    template void launch_energy<T>(const LatTable&, const T*, DevState, hipStream_t, bool, int);                    \
    template void launch_export<T>(const LatTable&, int, const T*, DevState, T*, hipStream_t);                 \
    template void launch_import<T>(const LatTable&, int, T*, DevState, const T*, hipStream_t);                 \
    template void launch_test_vonmises<T>(long, double, uint32_t, uint32_t, uint32_t, uint32_t, uint32_t, double*, \
                                          int*, hipStream_t);
LLR_INST(float)
LLR_INST(double)
#undef LLR_INST

}  // namespace llr
