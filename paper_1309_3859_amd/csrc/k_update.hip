// k_update.hip -- link initialisation and the checkerboard link update.
//
// Paper: Amado, Cardoso, Bicudo, arXiv 1309.3859, Sec. II (Wilson action,
// local updates with 3 overrelaxation steps), Sec. II.C.1 and Algorithm 1
// (sublattice updates with frozen boundary spatial links), Sec. II.D (links
// as phases, even then odd sites, in place).
//
// One work-item per link of the phase (direction mu, parity p, not frozen),
// every ensemble of the batch in the same launch: work-group b reads its time
// slice, its stretch of that slice and the geometry from one
// record (UpdBlock), the records dealt to the 8 XCDs in contiguous stretches
// and, within an ensemble, ordered time slice fastest (set by the host); where
// slices are short, a work-group holds several of them (SpanBlock).
// The staple of a link reads 18 angles: 12 of the other parity (coalesced,
// shifted by one site), 6 of the same parity; none of them is written by the
// phase, so the update is in place.  The all-link kernels below (start,
// health check, canonical gather and scatter, plaquettes) find their ensemble
// from block start offsets or a fixed number of blocks per ensemble.
#include <hip/hip_ext.h>

#include <mutex>
#include <type_traits>

#include "link_update.hpp"
#include "u1ml_internal.hpp"

namespace u1ml {

__device__ inline int find_ens(const int* __restrict__ bstart, int n_ens, int bid)
{
    int e = 0;
    while (e + 1 < n_ens && bid >= bstart[e + 1]) ++e;
    return e;
}

template <typename real>
struct LinkView {
    const real* base;
    int vh, nxh, ny, nz;
    __device__ inline real ld(int dir, int par, Coord c) const
    {
        const int h = (c.x >> 1) + nxh * (c.y + ny * (c.z + nz * c.t));
        return base[(size_t)(dir * 2 + par) * vh + h];
    }
};

// Byte offsets, within a time slice of one (direction, parity) array, of a
// site and its six spatial neighbours, for the link whose site has half index
// i in the slice (xh + Nx/2 (y + Ny z), x = 2 xh + odd).  The x step of an odd
// (even) x crosses to the next (previous) half index or stays; the others move
// by whole rows.  Offsets are those of the neighbour, so two of them combine
// as p + m - c.
template <typename real>
struct SliceNb {
    unsigned c, p[3], m[3];
    int odd_mask;  // all ones where x is odd

    // work-item tid of work-group record B, link parity par
    __device__ inline SliceNb(const UpdBlock& B, int tid, int par)
    {
        constexpr int w = sizeof(real);
        const int rx = B.x0 + tid;
        const int row = fdiv_small(rx, B.inv_nxh);
        const int xh = rx - __mul24(row, B.nxh);
        const int ry = B.y0 + row;
        const int dz = fdiv_small(ry, B.inv_ny);
        const int y = ry - __mul24(dz, B.ny);
        odd_mask = ((B.zt + par + y + dz) << 31) >> 31;
        const int sy = B.nxh * w, sz = sy * B.ny, st = B.slice * w;
        const int v = (B.i0 + tid) * w;
        c = (unsigned)v;
        p[0] = (unsigned)(v + (odd_mask & (xh == B.nxh - 1 ? w - sy : w)));
        m[0] = (unsigned)(v + (~odd_mask & (xh == 0 ? sy - w : -w)));
        p[1] = (unsigned)(v + (y == B.ny - 1 ? sy - sz : sy));
        m[1] = (unsigned)(v + (y == 0 ? sz - sy : -sy));
        p[2] = (unsigned)(v + (v >= st - sz ? sz - st : sz));
        m[2] = (unsigned)(v + (v < sz ? st - sz : -sz));
    }
};

// The six angles of the two staples of link (x, MU) in the plane (MU, NU):
//   v[0..2] = th_nu(x+mu), th_mu(x+nu), th_nu(x)          (forward)
//   v[3..5] = th_nu(x-nu), th_nu(x+mu-nu), th_mu(x-nu)    (backward)
// for a link of parity p in time slice t0 (byte offsets t0, tp, tm of the
// slice and its neighbours); vhb bytes per (direction, parity) array, src the
// byte offset of each direction's current buffer.
template <typename real, int MU, int NU>
__device__ inline void gather_slice(const LinkBuf<real>& lb, unsigned vhb, const unsigned* src, unsigned t0, unsigned tp,
                                    unsigned tm, const SliceNb<real>& nb, int p, real* v)
{
    const unsigned pp = (unsigned)p * vhb, pq = vhb - pp;
    const unsigned nu_p = NU * 2 * vhb + pp + src[NU], nu_q = NU * 2 * vhb + pq + src[NU];
    const unsigned mu_q = MU * 2 * vhb + pq + src[MU];
    // slice and offset of x + mu, x + nu, x - nu, x + mu - nu
    const unsigned s_pm = MU == 3 ? tp : t0, s_pn = NU == 3 ? tp : t0, s_mn = NU == 3 ? tm : t0;
    const unsigned s_pmmn = MU == 3 ? tp : (NU == 3 ? tm : t0);
    const unsigned o_pm = MU == 3 ? nb.c : nb.p[MU % 3], o_pn = NU == 3 ? nb.c : nb.p[NU % 3];
    const unsigned o_mn = NU == 3 ? nb.c : nb.m[NU % 3];
    const unsigned o_pmmn = MU == 3 ? o_mn : (NU == 3 ? o_pm : o_pm + (o_mn - nb.c));
    v[0] = lb.ld(o_pm, nu_q + s_pm);
    v[1] = lb.ld(o_pn, mu_q + s_pn);
    v[2] = lb.ld(nb.c, nu_p + t0);
    v[3] = lb.ld(o_mn, nu_q + s_mn);
    v[4] = lb.ld(o_pmmn, nu_p + s_pmmn);
    v[5] = lb.ld(o_mn, mu_q + s_mn);
}

// Byte offsets of work-item tid's site and its neighbours for a work-group over
// several time slices: t differs within a wave, so it is part of the offsets.
template <typename real>
struct SpanSite : SiteNb {
    int odd_mask;  // all ones where x is odd

    __device__ inline SpanSite(const SpanBlock& B, int tid, int par)
    {
        constexpr int w = sizeof(real);
        const int j = B.i0 + tid;
        const int ks = B.slice >= 1024 ? (int)(j >= B.slice) : fdiv_small(j, B.inv_slice);
        const int i = j - ks * B.slice;
        const int t = B.t0 + ks + (B.m ? (B.r0 + ks) / B.m : 0);
        const int row = fdiv(i, B.nxh, B.inv_nxh), xh = i - row * B.nxh;
        const int z = fdiv(row, B.ny, B.inv_ny), y = row - z * B.ny;
        odd_mask = -((t + par + y + z) & 1);
        const int sy = B.nxh * w, sz = sy * B.ny, st = B.slice * w, v = i * w;
        const unsigned at = (unsigned)t * (unsigned)st;
        c = at + (unsigned)v;
        p[0] = c + (unsigned)(odd_mask & (xh == B.nxh - 1 ? w - sy : w));
        m[0] = c + (unsigned)(~odd_mask & (xh == 0 ? sy - w : -w));
        p[1] = c + (unsigned)(y == B.ny - 1 ? sy - sz : sy);
        m[1] = c + (unsigned)(y == 0 ? sz - sy : -sy);
        p[2] = c + (unsigned)(v >= st - sz ? sz - st : sz);
        m[2] = c + (unsigned)(v < sz ? st - sz : -sz);
        p[3] = t == B.nt - 1 ? (unsigned)v : c + (unsigned)st;
        m[3] = t == 0 ? (unsigned)(B.nt - 1) * (unsigned)st + (unsigned)v : c - (unsigned)st;
    }
};

// One work-item per link of one checkerboard phase.  What bounds it: memory on
// lattices beyond the caches, launch and instruction latency on small ones (a
// dependent launch costs 1.85 us with 18 loads and a store in it; each further
// dependent instruction 2 to 3 ns).  So the index arithmetic is kept short: a
// work-group lies in one time slice, t and everything that follows from it is
// scalar, and the vector part of an address is one byte offset within the
// slice.
// WG: the heatbath's pending links are finished by work-group instead of by
// wave (hb_retry_wg).
// SPAN: a work-group goes on into the next time slices (SpanBlock), where slices
// do not fill whole waves.
template <typename real, int KIND, int MU, bool WG, bool SPAN>
__global__ void __launch_bounds__(1024)
    k_update(const EnsDesc* __restrict__ ens, const std::conditional_t<SPAN, SpanBlock, UpdBlock>* __restrict__ blocks,
             real* __restrict__ links, const uint32_t* __restrict__ upd, int pass_offset, int parity, unsigned src0,
             unsigned src1, unsigned src2, unsigned src3, double metro_delta)
{
    constexpr unsigned w = sizeof(real);
    extern __shared__ __align__(16) unsigned char queue_bytes[];
    // the whole record before the first branch: its loads are one round trip
    auto B = blocks[blockIdx.x];
    int n;
    if constexpr (SPAN) {
        asm volatile("" : "+s"(B.i0), "+s"(B.t0), "+s"(B.nxh), "+s"(B.inv_nxh), "+s"(B.link_off));
        n = B.n;
    } else {
        asm volatile("" : "+s"(B.i0), "+s"(B.x0), "+s"(B.t0), "+s"(B.nxh), "+s"(B.inv_nxh), "+s"(B.link_off));
        n = B.slice - B.i0;
    }
    const EnsDesc& E = ens[B.e];
    const int tid = (int)threadIdx.x;
    if ((WG ? 0 : tid & ~63) >= n) return;  // no link in this wave (work-group)
    const bool active = tid < n;
    const std::conditional_t<SPAN, SpanSite<real>, SliceNb<real>> nb(B, active ? tid : 0, parity);
    const LinkBuf<real> lb(links + B.link_off);
    const unsigned vhb = (unsigned)B.vh * w;
    const unsigned src[4] = {src0, src1, src2, src3};

    // every load of the update is issued before any arithmetic
    real v[3][6];
    unsigned self = (MU * 2 + (unsigned)parity) * vhb + src[MU];
    uint32_t half;  // half index of the link's site
    if constexpr (SPAN) {
        gather_nb<real, MU, Nu<MU, 0>::v, false>(lb, vhb, src, nb, parity, v[0]);
        gather_nb<real, MU, Nu<MU, 1>::v, false>(lb, vhb, src, nb, parity, v[1]);
        gather_nb<real, MU, Nu<MU, 2>::v, false>(lb, vhb, src, nb, parity, v[2]);
        half = nb.c / w;
    } else {
        const unsigned t0 = B.t0 * w, tp = B.tp * w, tm = B.tm * w;
        gather_slice<real, MU, Nu<MU, 0>::v>(lb, vhb, src, t0, tp, tm, nb, parity, v[0]);
        gather_slice<real, MU, Nu<MU, 1>::v>(lb, vhb, src, t0, tp, tm, nb, parity, v[1]);
        gather_slice<real, MU, Nu<MU, 2>::v>(lb, vhb, src, t0, tp, tm, nb, parity, v[2]);
        self += t0;
        half = (uint32_t)(B.i0 + tid) + B.t0;
    }
    real old = real(0);
    if (KIND != 0) old = lb.ld(nb.c, self);

    // the first Philox block depends only on the link's id and the counter:
    // formed here, it runs while the link angles are still in flight
    // canonical site x + Nx (y + Ny (z + Nz t)) = 2 half + odd
    const uint32_t lid = (uint32_t)MU + 8u * half + (nb.odd_mask & 4u);
    const uint32_t ctr = KIND == 1 ? 0u : upd[B.e] + (uint32_t)pass_offset;
    Block4 b0{};
    if (KIND != 1) b0 = philox4x32_10(lid, ctr, 0u, KIND == 2 ? DOM_METRO : DOM_HB, E.seed, E.key_id);

    if constexpr (WG) {
        real ar = real(0), ai = real(0), cp, sp;
        bool draw, pending;
        if (active) staple(v, &ar, &ai);
        const HbEnv<real> env = hb_first(active, b0, E.beta, &ar, ai, &cp, &sp, &draw, &pending);
        if (active && !pending) lb.st(hb_angle(ar, ai, cp, hb_sin(draw, cp, sp)), nb.c, self);
        int* counts = reinterpret_cast<int*>(queue_bytes);
        hb_retry_wg<real>(reinterpret_cast<HbWgQ<real>*>(queue_bytes + 64), counts, pending, env, lid, ar, ai, nb.c, ctr,
                          E.seed, E.key_id, [&](real th, unsigned off) { lb.st(th, off, self); },
                          [&](unsigned off) { return lb.ld(off, self); });
    } else {
        HbQ<real>* wave_q = reinterpret_cast<HbQ<real>*>(queue_bytes) + (tid & ~63);
        const real th = update_link<real, KIND>(active, v, b0, lid, ctr, E.beta, E.seed, E.key_id, metro_delta, wave_q,
                                                [&] { return KIND == 0 ? lb.ld(nb.c, self) : old; });
        if (active) lb.st(th, nb.c, self);
    }
}

// With a start/stop event pair the launch goes through hipExtLaunchKernelGGL,
// whose events take the dispatch's own begin and end timestamps.
template <typename real, int KIND, int MU, bool WG, bool SPAN>
static void launch_update_mu(const UpdLaunch& a)
{
    const dim3 g(a.total_blocks), b(a.block);
    const size_t lds = KIND != 0 ? 0 : (WG ? 64 + sizeof(HbWgQ<real>) * b.x : sizeof(HbQ<real>) * b.x);
    const auto* blocks = reinterpret_cast<const std::conditional_t<SPAN, SpanBlock, UpdBlock>*>(a.d_blocks);
    if (a.ev_start)
        hipExtLaunchKernelGGL((k_update<real, KIND, MU, WG, SPAN>), g, b, lds, a.st, a.ev_start, a.ev_stop, 0, a.d_ens,
                              blocks, (real*)a.links, a.d_upd, a.pass_offset, a.parity, a.src[0], a.src[1],
                              a.src[2], a.src[3], a.metro_delta);
    else
        hipLaunchKernelGGL((k_update<real, KIND, MU, WG, SPAN>), g, b, lds, a.st, a.d_ens, blocks, (real*)a.links,
                           a.d_upd, a.pass_offset, a.parity, a.src[0], a.src[1], a.src[2], a.src[3], a.metro_delta);
}

template <typename real, int KIND, bool WG, bool SPAN>
static void launch_update_t(const UpdLaunch& a)
{
    switch (a.mu) {
    case 0: launch_update_mu<real, KIND, 0, WG, SPAN>(a); break;
    case 1: launch_update_mu<real, KIND, 1, WG, SPAN>(a); break;
    case 2: launch_update_mu<real, KIND, 2, WG, SPAN>(a); break;
    default: launch_update_mu<real, KIND, 3, WG, SPAN>(a); break;
    }
}

// Launches of at least this many work-groups finish the heatbath's pending
// links by work-group: where the vector units are the bound, the rounds saved
// outweigh the barrier.  Wave by wave / by work-group: 3 sweeps of 128^3 x 16
// FP32 (65,536 work-groups) 13.49 / 13.14 ms, 48^3 x 12 FP32 (2,592) 70.5 / 70.9,
// 16 ensembles FP32 (about 1,000 a lane) 8.76 / 8.81, FP64 19.05 / 18.56, 24^3 x 8
// FP64 (216) 14.8 / 16.3.
template <typename real>
constexpr int kHbWgBlocks = sizeof(real) == 8 ? 640 : 4096;

template <typename real, bool SPAN>
static void launch_update_r(const UpdLaunch& a)
{
    const bool wg = a.total_blocks >= kHbWgBlocks<real> && a.block <= 512;
    switch (a.kind) {
    case 0: wg ? launch_update_t<real, 0, true, SPAN>(a) : launch_update_t<real, 0, false, SPAN>(a); break;
    case 1: launch_update_t<real, 1, false, SPAN>(a); break;
    default: launch_update_t<real, 2, false, SPAN>(a); break;
    }
}

hipError_t launch_update(const UpdLaunch& a)
{
    if (a.total_blocks <= 0) return hipSuccess;
    if ((a.ev_start == nullptr) != (a.ev_stop == nullptr) || a.kind < 0 || a.kind > 2) return hipErrorInvalidValue;
    if (a.precision == 0)
        a.span ? launch_update_r<double, true>(a) : launch_update_r<double, false>(a);
    else
        a.span ? launch_update_r<float, true>(a) : launch_update_r<float, false>(a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// All-link kernels: one work-item per (direction, parity, half site).
// ---------------------------------------------------------------------------
struct LinkItem {
    int dir, par, h, x, y, z, t;
};

__device__ inline bool decode_link(const EnsDesc& E, int item, LinkItem* o)
{
    if (item >= 8 * E.vh) return false;
    const int dp = item / E.vh;
    o->h = item - dp * E.vh;
    o->dir = dp >> 1;
    o->par = dp & 1;
    const int row = o->h / E.nxh;
    const int xh = o->h - row * E.nxh;
    const int yz = row;
    o->t = yz / (E.ny * E.nz);
    const int r2 = yz - o->t * E.ny * E.nz;
    o->z = r2 / E.ny;
    o->y = r2 - o->z * E.ny;
    o->x = 2 * xh + ((o->y + o->z + o->t + o->par) & 1);
    return true;
}

// Cold: theta = 0.  Hot: theta = pi (2u - 1), u = (w0 + 1/2) 2^-32 with w0 the
// first word of the Philox block (link id, 0, 0, INIT); formed in FP64 and
// rounded to the storage precision.
template <typename real>
__global__ void k_init(const EnsDesc* __restrict__ ens, const int* __restrict__ bstart, int n_ens,
                       real* __restrict__ links, int start)
{
    const int bid = blockIdx.x;
    const int e = find_ens(bstart, n_ens, bid);
    const EnsDesc& E = ens[e];
    LinkItem it;
    if (!decode_link(E, (bid - bstart[e]) * (int)blockDim.x + (int)threadIdx.x, &it)) return;
    double th = 0.0;
    if (start) {
        const uint32_t lid = (uint32_t)(it.dir + 4 * (it.x + E.nx * (it.y + E.ny * (it.z + E.nz * it.t))));
        const Block4 b = philox4x32_10(lid, 0u, 0u, DOM_INIT, E.seed, E.key_id);
        const double u = ((double)b.w[0] + 0.5) * (1.0 / 4294967296.0);
        th = M<double>::pi * (2.0 * u - 1.0);
    }
    links[E.link_off + (size_t)(it.dir * 2 + it.par) * E.vh + it.h] = (real)th;
}

hipError_t launch_init_links(const EnsDesc* d_ens, const int* d_bstart_all, int n_ens, int total_blocks, int precision,
                             void* links, int start, hipStream_t st)
{
    if (precision == 0)
        hipLaunchKernelGGL(k_init<double>, dim3(total_blocks), dim3(256), 0, st, d_ens, d_bstart_all, n_ens,
                           (double*)links, start);
    else
        hipLaunchKernelGGL(k_init<float>, dim3(total_blocks), dim3(256), 0, st, d_ens, d_bstart_all, n_ens,
                           (float*)links, start);
    return hipGetLastError();
}

template <typename real>
__global__ void k_health(const EnsDesc* __restrict__ ens, const int* __restrict__ bstart, int n_ens,
                         const real* __restrict__ links, unsigned long long* __restrict__ count)
{
    const int bid = blockIdx.x;
    const int e = find_ens(bstart, n_ens, bid);
    const EnsDesc& E = ens[e];
    LinkItem it;
    if (!decode_link(E, (bid - bstart[e]) * (int)blockDim.x + (int)threadIdx.x, &it)) return;
    const double th = (double)links[E.link_off + (size_t)(it.dir * 2 + it.par) * E.vh + it.h];
    const double lim = M<double>::pi * (1.0 + 1.0 / 1048576.0);
    if (!(th >= -lim && th <= lim)) atomicAdd(count, 1ull);
}

hipError_t launch_health(const EnsDesc* d_ens, const int* d_bstart_all, int n_ens, int total_blocks, int precision,
                         const void* links, unsigned long long* d_count, hipStream_t st)
{
    if (precision == 0)
        hipLaunchKernelGGL(k_health<double>, dim3(total_blocks), dim3(256), 0, st, d_ens, d_bstart_all, n_ens,
                           (const double*)links, d_count);
    else
        hipLaunchKernelGGL(k_health<float>, dim3(total_blocks), dim3(256), 0, st, d_ens, d_bstart_all, n_ens,
                           (const float*)links, d_count);
    return hipGetLastError();
}

// Canonical FP64 view <-> even/odd storage, one ensemble at a time.
template <typename real>
__global__ void k_gather(const EnsDesc* __restrict__ ens, int e, const real* __restrict__ links,
                         double* __restrict__ canon, long long n_sites)
{
    const long long s = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n_sites) return;
    const EnsDesc& E = ens[e];
    const int x = (int)(s % E.nx);
    long long r = s / E.nx;
    const int y = (int)(r % E.ny);
    r /= E.ny;
    const int z = (int)(r % E.nz);
    const int t = (int)(r / E.nz);
    const int par = (x + y + z + t) & 1;
    const int h = (x >> 1) + E.nxh * (y + E.ny * (z + E.nz * t));
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) canon[4 * s + mu] = (double)links[E.link_off + (size_t)(mu * 2 + par) * E.vh + h];
}

template <typename real>
__global__ void k_scatter(const EnsDesc* __restrict__ ens, int e, real* __restrict__ links,
                          const double* __restrict__ canon, long long n_sites)
{
    const long long s = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n_sites) return;
    const EnsDesc& E = ens[e];
    const int x = (int)(s % E.nx);
    long long r = s / E.nx;
    const int y = (int)(r % E.ny);
    r /= E.ny;
    const int z = (int)(r % E.nz);
    const int t = (int)(r / E.nz);
    const int par = (x + y + z + t) & 1;
    const int h = (x >> 1) + E.nxh * (y + E.ny * (z + E.nz * t));
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) links[E.link_off + (size_t)(mu * 2 + par) * E.vh + h] = (real)canon[4 * s + mu];
}

hipError_t launch_gather_links(const EnsDesc* d_ens, int ens, int precision, const void* links, double* d_canon,
                               long long n_sites, hipStream_t st)
{
    const int g = (int)((n_sites + 255) / 256);
    if (precision == 0)
        hipLaunchKernelGGL(k_gather<double>, dim3(g), dim3(256), 0, st, d_ens, ens, (const double*)links, d_canon,
                           n_sites);
    else
        hipLaunchKernelGGL(k_gather<float>, dim3(g), dim3(256), 0, st, d_ens, ens, (const float*)links, d_canon,
                           n_sites);
    return hipGetLastError();
}

hipError_t launch_scatter_links(const EnsDesc* d_ens, int ens, int precision, void* links, const double* d_canon,
                                long long n_sites, hipStream_t st)
{
    const int g = (int)((n_sites + 255) / 256);
    if (precision == 0)
        hipLaunchKernelGGL(k_scatter<double>, dim3(g), dim3(256), 0, st, d_ens, ens, (double*)links, d_canon,
                           n_sites);
    else
        hipLaunchKernelGGL(k_scatter<float>, dim3(g), dim3(256), 0, st, d_ens, ens, (float*)links, d_canon, n_sites);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Plaquette means per orientation (E_x, E_y, E_z, B_x, B_y, B_z), FP64 sums.
// Work-group (e, b), one of kPlaqBlocks per ensemble, walks the ensemble's
// sites in a fixed stride (V < 2^28 sites, so 32-bit indices) and reduces its
// sums through LDS; k_plaq_final adds an ensemble's partials in a fixed-order
// tree.
// ---------------------------------------------------------------------------
template <typename real>
__global__ void __launch_bounds__(256) k_plaq_partial(const EnsDesc* __restrict__ ens, const real* __restrict__ links,
                                                      double* __restrict__ partials)
{
    const int e = blockIdx.x / kPlaqBlocks;
    const int b = blockIdx.x % kPlaqBlocks;
    const EnsDesc& E = ens[e];
    LinkView<real> L{links + E.link_off, E.vh, E.nxh, E.ny, E.nz};
    const int V = 2 * E.vh;
    double acc[6] = {0, 0, 0, 0, 0, 0};
    static const int pa[6] = {0, 1, 2, 1, 2, 0};
    static const int pb[6] = {3, 3, 3, 2, 0, 1};
    for (int s = b * 256 + (int)threadIdx.x; s < V; s += 256 * kPlaqBlocks) {
        const int x = s % E.nx;
        int r = s / E.nx;
        const int y = r % E.ny;
        r /= E.ny;
        const int z = r % E.nz;
        const int t = r / E.nz;
        const Coord c = {x, y, z, t};
        const int p = (x + y + z + t) & 1;
#pragma unroll
        for (int o = 0; o < 6; ++o) {
            const int a = pa[o], bb = pb[o];
            const Coord ca = step(c, a, +1, E.nx, E.ny, E.nz, E.nt);
            const Coord cb = step(c, bb, +1, E.nx, E.ny, E.nz, E.nt);
            const double th = (double)L.ld(a, p, c) + (double)L.ld(bb, p ^ 1, ca) - (double)L.ld(a, p ^ 1, cb) -
                              (double)L.ld(bb, p, c);
            acc[o] += cos(th);
        }
    }
    __shared__ double sh[6][256];
    for (int o = 0; o < 6; ++o) sh[o][threadIdx.x] = acc[o];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int o = 0; o < 6; ++o) sh[o][threadIdx.x] += sh[o][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x < 6) partials[(size_t)blockIdx.x * 6 + threadIdx.x] = sh[threadIdx.x][0];
}

// one 256-thread work-group per ensemble: thread i adds partials i, i + 256,
// ... in order, then an LDS tree
__global__ void __launch_bounds__(256) k_plaq_final(const EnsDesc* __restrict__ ens,
                                                    const double* __restrict__ partials, double* __restrict__ out)
{
    const int e = blockIdx.x;
    double acc[6] = {0, 0, 0, 0, 0, 0};
    for (int b = threadIdx.x; b < kPlaqBlocks; b += blockDim.x)
        for (int o = 0; o < 6; ++o) acc[o] += partials[((size_t)e * kPlaqBlocks + b) * 6 + o];
    __shared__ double sh[6][256];
    for (int o = 0; o < 6; ++o) sh[o][threadIdx.x] = acc[o];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int o = 0; o < 6; ++o) sh[o][threadIdx.x] += sh[o][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x < 6) out[e * 6 + threadIdx.x] = sh[threadIdx.x][0] / (2.0 * (double)ens[e].vh);
}

hipError_t launch_plaquette(const EnsDesc* d_ens, int n_ens, int, int precision, const void* links,
                            double* d_partials, double* d_out, hipStream_t st)
{
    if (precision == 0)
        hipLaunchKernelGGL(k_plaq_partial<double>, dim3(n_ens * kPlaqBlocks), dim3(256), 0, st, d_ens,
                           (const double*)links, d_partials);
    else
        hipLaunchKernelGGL(k_plaq_partial<float>, dim3(n_ens * kPlaqBlocks), dim3(256), 0, st, d_ens,
                           (const float*)links, d_partials);
    hipLaunchKernelGGL(k_plaq_final, dim3(n_ens), dim3(256), 0, st, d_ens, d_partials, d_out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Static scratch of the allocation-free plaquette call: the per-work-group
// partial sums of up to kStaticPlaqEns ensembles (1.5 MiB), one copy per
// device for the life of the process.  Host code must not pass the array's
// name to a kernel: it reaches the array only through the address that
// hipGetSymbolAddress returns with the device current, kept per device.
// ---------------------------------------------------------------------------
static __device__ __align__(256) double scratch[(size_t)kStaticPlaqEns * kPlaqBlocks * 6];

hipError_t static_scratch(double** ptr)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static double* addr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[dev] = static_cast<double*>(p);
    }
    *ptr = addr[dev];
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// RNG and sampler fills (bit-exact and statistical checks of the stream).
// ---------------------------------------------------------------------------
__global__ void k_philox_fill(uint32_t k0, uint32_t k1, uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, size_t n,
                              uint32_t* __restrict__ out)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const Block4 b = philox4x32_10(c0 + (uint32_t)i, c1, c2, c3, k0, k1);
    uint4 v;
    v.x = b.w[0];
    v.y = b.w[1];
    v.z = b.w[2];
    v.w = b.w[3];
    reinterpret_cast<uint4*>(out)[i] = v;
}

hipError_t launch_philox_fill(uint32_t k0, uint32_t k1, uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, size_t n,
                              uint32_t* d_out, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_philox_fill, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, k0, k1, c0, c1, c2, c3, n,
                       d_out);
    return hipGetLastError();
}

template <typename real>
__global__ void k_vonmises_fill(real kappa, uint32_t seed, uint32_t key_id, uint32_t c0, uint32_t c1, size_t n,
                                double* __restrict__ out, int* __restrict__ att)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int na;
    const real psi = vonmises_psi<real>(kappa, seed, key_id, c0 + (uint32_t)i, c1, DOM_TEST, &na);
    out[i] = (double)psi;
    if (att) att[i] = na;
}

hipError_t launch_vonmises_fill(double kappa, int precision, uint32_t seed, uint32_t key_id, uint32_t c0, uint32_t c1,
                                size_t n, double* d_out, int* d_att, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    const dim3 g((unsigned)((n + 255) / 256));
    if (precision == 0)
        hipLaunchKernelGGL(k_vonmises_fill<double>, g, dim3(256), 0, st, kappa, seed, key_id, c0, c1, n, d_out, d_att);
    else
        hipLaunchKernelGGL(k_vonmises_fill<float>, g, dim3(256), 0, st, (float)kappa, seed, key_id, c0, c1, n, d_out,
                           d_att);
    return hipGetLastError();
}

// the library's FP64 sine and cosine on given arguments
__global__ void k_sincos_fill(const double* __restrict__ x, size_t n, double* __restrict__ s, double* __restrict__ c)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double sv, cv;
    sincos_bounded(x[i], &sv, &cv);
    s[i] = sv;
    c[i] = cv;
}

hipError_t launch_sincos_fill(const double* d_x, size_t n, double* d_s, double* d_c, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_sincos_fill, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, d_x, n, d_s, d_c);
    return hipGetLastError();
}

// advances the counters of the n_ens ensembles described by ens[]
__global__ void k_advance(const EnsDesc* __restrict__ ens, uint32_t* __restrict__ upd, int n_ens, int delta)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n_ens) upd[ens[e].res_index] += (uint32_t)delta;
}

hipError_t launch_advance_counters(const EnsDesc* d_ens, uint32_t* d_upd, int n_ens, int delta, hipStream_t st)
{
    hipLaunchKernelGGL(k_advance, dim3((n_ens + 63) / 64), dim3(64), 0, st, d_ens, d_upd, n_ens, delta);
    return hipGetLastError();
}

}  // namespace u1ml
