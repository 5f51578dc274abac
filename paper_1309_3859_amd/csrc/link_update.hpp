// link_update.hpp -- one link's update (heatbath, overrelaxation, Metropolis)
// from its staple angles, shared by the kernels that visit the links.
//
// Paper: Amado, Cardoso, Bicudo, arXiv 1309.3859, Sec. II.
#pragma once

#include "device_common.hpp"

namespace u1ml {

// ---------------------------------------------------------------------------
// Addresses.  The links of one ensemble span less than 4 GiB: they are read
// and written through a buffer resource, one 32-bit scalar offset naming the
// (direction, parity) array and the time slice, one 32-bit vector offset the
// site, so that an address costs one scalar addition and no vector one.
// ---------------------------------------------------------------------------
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

template <typename real>
struct LinkBuf {
    __amdgpu_buffer_rsrc_t rsrc;
    __device__ inline explicit LinkBuf(real* base)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc(base, 0, 0xFFFFFFFFu, 0x00020000))
    {
    }
    __device__ inline real ld(unsigned voff, unsigned soff) const
    {
        if constexpr (sizeof(real) == 8)
            return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rsrc, voff, soff, 0));
        else
            return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, voff, soff, 0));
    }
    __device__ inline void st(real v, unsigned voff, unsigned soff) const
    {
        if constexpr (sizeof(real) == 8)
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), rsrc, voff, soff, 0);
        else
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), rsrc, voff, soff, 0);
    }
};

// Byte offsets of a site and its eight neighbours within one (direction,
// parity) array.
struct SiteNb {
    unsigned c, p[4], m[4];
};

// The angles of the two staples of link (x, MU) in the plane (MU, NU), as the
// one-parity kernel names them; SKIP: not th_mu(x +- nu) (v[1] and v[5]).
template <typename real, int MU, int NU, bool SKIP>
__device__ inline void gather_nb(const LinkBuf<real>& lb, unsigned vhb, const unsigned* src, const SiteNb& nb, int p,
                                 real* v)
{
    const unsigned pp = (unsigned)p * vhb, pq = vhb - pp;
    const unsigned nu_p = NU * 2 * vhb + pp + src[NU], nu_q = NU * 2 * vhb + pq + src[NU];
    const unsigned mu_q = MU * 2 * vhb + pq + src[MU];
    v[0] = lb.ld(nb.p[MU], nu_q);
    if (!SKIP) v[1] = lb.ld(nb.p[NU], mu_q);
    v[2] = lb.ld(nb.c, nu_p);
    v[3] = lb.ld(nb.m[NU], nu_q);
    v[4] = lb.ld(nb.p[MU] + (nb.m[NU] - nb.c), nu_p);
    if (!SKIP) v[5] = lb.ld(nb.m[NU], mu_q);
}

// Quotient a / b of a small index by an extent: 0 <= a < b + 2^10 and b <=
// 2^22, or a < 2^21; inv_b = 1/b rounded.  (a + 1/2) / b lies at least 1/(2b) from an
// integer, further than the rounding of the reciprocal and of the one product,
// so no correction step is needed.
__device__ inline int fdiv_small(int a, float inv_b) { return (int)(((float)a + 0.5f) * inv_b); }

// ---------------------------------------------------------------------------
// Heatbath draws.  A deviate is returned as (c, s): FP32 cos psi and sin psi,
// FP64 cos psi and the sign of sin psi (the sine is formed once, by hb_angle's
// caller).
// ---------------------------------------------------------------------------
template <typename real>
struct HbEnv;
template <>
struct HbEnv<float> {
    BfEnvF32 v;
    __device__ inline explicit HbEnv(float kappa) : v(bf_env_f32(kappa)) {}
};
template <>
struct HbEnv<double> {
    double kappa, r;
    __device__ inline explicit HbEnv(double k) : kappa(k), r(bf_r_f64(k)) {}
    __device__ inline HbEnv(double k, double rr) : kappa(k), r(rr) {}
};

// the two attempts of one Philox block; true if one accepted
__device__ inline bool hb_try(const HbEnv<float>& e, const Block4& b, float* c, float* s)
{
    return bf_pair_f32(e.v, b, c, s) != 0;
}
__device__ inline bool hb_try(const HbEnv<double>& e, const Block4& b, double* c, double* s)
{
    bool neg;
    if (!bf_pair_f64(e.kappa, e.r, b, c, &neg)) return false;
    *s = neg ? -1.0 : 1.0;
    return true;
}

// A pending link's entry in its wave's LDS queue: what further attempts need,
// then the deviate (c = 2: none of the attempts accepted).
template <typename real>
struct HbQ;
template <>
struct HbQ<float> {
    float a, b;  // kappa, link id; c, s
    __device__ inline void put(const HbEnv<float>& e, uint32_t lid) { a = e.v.kappa, b = __uint_as_float(lid); }
    __device__ inline HbEnv<float> env() const { return HbEnv<float>(a); }
    __device__ inline uint32_t lid() const { return __float_as_uint(b); }
};
template <>
struct HbQ<double> {
    double a, b, id;  // kappa, r, link id; c, s
    __device__ inline void put(const HbEnv<double>& e, uint32_t lid)
    {
        a = e.kappa, b = e.r, id = __longlong_as_double((long long)lid);
    }
    __device__ inline HbEnv<double> env() const { return HbEnv<double>(a, b); }
    __device__ inline uint32_t lid() const { return (uint32_t)__double_as_longlong(id); }
};

__device__ inline void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// theta = arg(e^{i psi} conj A): one atan2 for wrap(psi - arg A), in [-pi, pi)
__device__ inline float hb_angle(float ar, float ai, float cp, float sp)
{
    const float th = atan2_fast(sp * ar - cp * ai, cp * ar + sp * ai);
    return th >= 3.14159265f ? -3.14159265f : th;
}
__device__ inline double hb_angle(double ar, double ai, double cp, double sp)
{
    const double th = M<double>::atan2_(sp * ar - cp * ai, cp * ar + sp * ai);
    return th >= M<double>::pi ? -M<double>::pi : th;
}

// sin psi of an accepted deviate (c, s), or of the uniform psi (s itself)
__device__ inline float hb_sin(bool, float, float s) { return s; }
__device__ inline double hb_sin(bool draw, double c, double s)
{
    if (!draw) return s;
    // +-sqrt((1 - f)(1 + f)) (1 - f and 1 + f exact where they cancel)
    const double sq = M<double>::sqrt_((1.0 - c) * (1.0 + c));
    return s < 0.0 ? -sq : sq;
}

// One round after another of further Philox blocks (1 .. 32767, attempts 2 ..
// 65535) for the links dealt to a wave, 2^lg consecutive lanes each: a round
// tries 2^lg blocks of every link at once and the first accepting block in
// attempt order decides, so the result is that of trying them one after
// another.  take(c, s) is called once per link, by one of its lanes; links
// that never accept call it with c = 2.
template <typename real, typename Take>
__device__ inline void hb_rounds(bool open, int lg, const HbEnv<real>& env, uint32_t lid, uint32_t ctr, uint32_t seed,
                                 uint32_t key, Take take)
{
    const int lane = threadIdx.x & 63, sub = lane & ((1 << lg) - 1);
    const unsigned long long gm = (lg == 6 ? ~0ull : (1ull << (1 << lg)) - 1ull) << (lane - sub);
    for (uint32_t j0 = 1; j0 < 32768u && __any(open); j0 += 1u << lg) {
        const uint32_t jp = j0 + (uint32_t)sub;
        real c = real(0), s = real(0);
        bool ok = open && jp < 32768u;
        if (ok) ok = hb_try(env, philox4x32_10(lid, ctr, jp, DOM_HB, seed, key), &c, &s);
        const unsigned long long hit = __ballot(ok) & gm;
        if (hit) {
            if (lane == __ffsll(hit) - 1) take(c, s);
            open = false;
        }
    }
    if (open && sub == 0) take(real(2), real(0));
}

// The wave's pending links (about 1 in 12) after the first block: its lanes are
// dealt to them, with the usual 5 pending links 8 blocks (16 attempts) of each
// in a round, so one round is enough, where one lane per link over the whole
// work-group took three serial rounds between two barriers.  (Four attempts by
// every lane before this step measured slower: 24^3 x 8 sweeps 89 instead of 88
// us, the FP64 batch of 16 ensembles 22.7 instead of 21.9 ms.)  Called by whole
// waves.
template <typename real>
__device__ inline void hb_retry(HbQ<real>* q, bool pending, const HbEnv<real>& mine, uint32_t lid, uint32_t ctr,
                                uint32_t seed, uint32_t key, real* c, real* s)
{
    const unsigned long long m = __ballot(pending);
    if (m == 0) return;  // uniform
    const int lane = threadIdx.x & 63;
    const int n = __popcll(m);
    const int rank = __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0));
    if (pending) q[rank].put(mine, lid);
    wave_lds_sync();
    const int lg = __clz(n - 1) - 26;  // floor(log2(64 / n))
    const int g = lane >> lg;
    const HbQ<real> r = q[g < n ? g : 0];
    hb_rounds<real>(g < n, lg, r.env(), r.lid(), ctr, seed, key, [&](real cc, real ss) { q[g].a = cc, q[g].b = ss; });
    wave_lds_sync();
    if (pending) *c = q[rank].a, *s = q[rank].b;
}

// A pending link's entry in its work-group's LDS queue: what further attempts
// and the new angle need.
template <typename real>
struct HbWgQ {
    HbQ<real> q;
    real ar, ai;
    unsigned off;  // the link's byte offset from the launch's link base
};

// The work-group's pending links: every wave leaves its own in its 64 entries,
// and after a barrier they are dealt to as few waves as hold them (one of four
// with work-groups of 256); the others are done.  Fewer rounds for the chip
// than wave by wave (a round costs a Philox block, 480 cycles of quarter-rate
// multiplications, and two attempts), one barrier more for each work-group, so
// large launches use it.  put(theta, off) stores a link's new angle;
// old(off) reads its old one.  Called by whole work-groups.
template <typename real, typename Put, typename Old>
__device__ inline void hb_retry_wg(HbWgQ<real>* queue, int* counts, bool pending, const HbEnv<real>& mine, uint32_t lid,
                                   real ar, real ai, unsigned off, uint32_t ctr, uint32_t seed, uint32_t key, Put put,
                                   Old old)
{
    const unsigned long long m = __ballot(pending);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    if (lane == 0) counts[wave] = __popcll(m);
    if (pending) {
        HbWgQ<real>& e = queue[(wave << 6) +
                               __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0))];
        e.q.put(mine, lid);
        e.ar = ar, e.ai = ai, e.off = off;
    }
    __syncthreads();
    int total = 0;
    for (int w = 0; w < nw; ++w) total += counts[w];
    total = __builtin_amdgcn_readfirstlane(total);
    // links 64 wave .. 64 wave + 63 of the work-group's pending ones
    const int n = min(total - (wave << 6), 64);
    if (n <= 0) return;  // uniform
    const int lg = __clz(n - 1) - 26;
    const int g = lane >> lg, k = (wave << 6) + (g < n ? g : 0);
    int slot = 0, base = 0;
    for (int w = 0; w < nw; ++w) {
        const int c = counts[w];
        if (k >= base && k < base + c) slot = (w << 6) + k - base;
        base += c;
    }
    const HbWgQ<real> e = queue[slot];
    hb_rounds<real>(g < n, lg, e.q.env(), e.q.lid(), ctr, seed, key, [&](real c, real s) {
        put(c == real(2) ? old(e.off) : hb_angle(e.ar, e.ai, c, hb_sin(true, c, s)), e.off);
    });
}

// Staple sum A = sum_{nu != mu} exp(i phi_f) + exp(i phi_b), nu ascending,
// forward before backward, phi_f = v0 - v1 - v2, phi_b = v3 - v4 - v5.
template <typename real>
__device__ inline void staple(const real (&v)[3][6], real* ar, real* ai)
{
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        real s, co;
        M<real>::sincos_(v[k][0] - v[k][1] - v[k][2], &s, &co);
        if (k == 0) {
            *ar = co;
            *ai = s;
        } else {
            *ar += co;
            *ai += s;
        }
        M<real>::sincos_(v[k][3] - v[k][4] - v[k][5], &s, &co);
        *ar += co;
        *ai += s;
    }
}

// A link's envelope and its first Philox block's attempts.  draw: kappa > 0
// (else psi is uniform, (c, s) its cosine and sine, and with A = 0 as well
// theta = psi, for which *ar becomes 1); pending: neither attempt accepted.
template <typename real>
__device__ inline HbEnv<real> hb_first(bool active, const Block4& b0, double beta, real* ar, real ai, real* cp, real* sp,
                                       bool* draw, bool* pending)
{
    using m = M<real>;
    real kappa = real(1);
    *cp = *sp = real(0);
    if (active) {
        const real R = m::sqrt_(*ar * *ar + ai * ai);
        kappa = (real)beta * R;
        if (kappa == real(0)) {
            // attempt 0: pi (2 U1 - 1)
            if (R == real(0)) *ar = real(1);
            if constexpr (sizeof(real) == 4) {
                const float rev = m::u1(b0.w[0]) - 0.5f;  // in revolutions
                *cp = __builtin_amdgcn_cosf(rev);
                *sp = __builtin_amdgcn_sinf(rev);
            } else {
                sincos_bounded(m::pi * (2.0 * m::u1(b0.w[0]) - 1.0), sp, cp);
            }
        }
    }
    *draw = active && kappa != real(0);
    const HbEnv<real> env(*draw ? kappa : real(1));
    *pending = false;
    if (*draw) *pending = !hb_try(env, b0, cp, sp);
    return env;
}

// ---------------------------------------------------------------------------
// One link's update from its 18 staple angles v, its old angle, its first
// Philox block, its id and the stochastic pass counter.  Staple sum A = sum_{nu != mu} exp(i phi_f) +
// exp(i phi_b), nu ascending, forward before backward, phi_f = v0 - v1 - v2,
// phi_b = v3 - v4 - v5.
// kind 0: heatbath theta = wrap(psi - arg A), psi ~ vonMises(0, beta |A|);
//         the old angle is asked for only if no attempt accepts;
// kind 1: overrelaxation theta = wrap(-theta - 2 arg A) (unchanged if A = 0);
// kind 2: Metropolis (the paper's update), one hit per link.
// Called by whole waves (active: this lane has a link).
// ---------------------------------------------------------------------------
template <typename real, int KIND, typename OldF>
__device__ inline real update_link(bool active, const real (&v)[3][6], const Block4& b0, uint32_t lid, uint32_t ctr,
                                   double beta, uint32_t seed, uint32_t key, double metro_delta, HbQ<real>* wave_q,
                                   OldF old_angle)
{
    using m = M<real>;
    real ar = real(0), ai = real(0), th = real(0);
    if (active) staple(v, &ar, &ai);
    if constexpr (KIND == 0) {
        real cp, sp;
        bool draw, pending;
        const HbEnv<real> env = hb_first(active, b0, beta, &ar, ai, &cp, &sp, &draw, &pending);
        hb_retry<real>(wave_q, pending, env, lid, ctr, seed, key, &cp, &sp);
        if (active) th = cp == real(2) ? old_angle() : hb_angle(ar, ai, cp, hb_sin(draw, cp, sp));
    } else if constexpr (KIND == 2) {
        // Metropolis: theta' = theta + delta (2 U1 - 1), accepted when
        // U2 < exp(beta (Re(e^{i theta'} A) - Re(e^{i theta} A)))
        if (active) {
            const real old = old_angle();
            const real thn = wrap_angle<real>(old + (real)metro_delta * (real(2) * m::u1(b0.w[0]) - real(1)));
            real sn, cn, so, co;
            m::sincos_(thn, &sn, &cn);
            m::sincos_(old, &so, &co);
            const real dl = (real)beta * ((ar * cn - ai * sn) - (ar * co - ai * so));
            th = (dl >= real(0) || m::u2(b0.w[1]) < m::exp_(dl)) ? thn : old;
        }
    } else {
        if (active) {
            const real old = old_angle();
            const real phiA = m::atan2_(ai, ar);
            th = wrap_angle<real>(-old - real(2) * phiA);
            if (ar == real(0) && ai == real(0)) th = old;
        }
    }
    return th;
}

}  // namespace u1ml
