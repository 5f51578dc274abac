// k_slab.hip -- whole sweeps of small lattices in one launch, links in LDS.
//
// Paper: Amado, Cardoso, Bicudo, arXiv 1309.3859, Sec. II (local updates with
// 3 overrelaxation steps), Sec. II.C.1 and Algorithm 1 (sublattice updates
// with frozen boundary spatial links: slabs do not see each other), Sec. II.D.
//
// One work-group owns one slab (or, with every link updated, one lattice): it
// copies the slab's links and the frozen spatial links of the layer above into
// LDS, runs n_sweeps sweeps of every direction and parity there with a barrier
// between phases, and copies the updated links back.  The same updates in the
// same order with the same Philox blocks as one launch per phase, so the same
// links, bit for bit.
//
// What bounds it: on one compute unit, the instruction chain of a phase (an
// overrelaxation about 0.4 us in FP32, 1 us in FP64) times its waves per SIMD,
// against 1.9 us and more for a launch.
#include "link_update.hpp"
#include "u1ml_internal.hpp"

namespace u1ml {

// Neighbours of a half index within its layer, as byte offsets in the layer:
// rows up (high half) and down (low half) in y and z, the next and previous
// half index in the row (periodic); parity of y + z.
struct SlabNb {
    unsigned y, z, x, par;
};

// The slab's links in LDS: one array per (direction, parity) as in memory,
// layer after layer; strides in bytes.
template <typename real>
struct SlabView {
    char* lds;
    int layer, par, dir;
    __device__ inline real& at(unsigned arr, unsigned off) const { return *reinterpret_cast<real*>(lds + arr + off); }
};

// Byte offsets of a site and its eight neighbours within one array.
struct SlabSite {
    unsigned c, p[4], m[4];
};

// The 18 staple angles of link (site, MU) of parity par, as the one-parity
// kernel names them.
template <typename real, int MU>
__device__ inline void gather_lds(const SlabView<real>& V, const SlabSite& s, int par, real (&v)[3][6])
{
    const unsigned pp = (unsigned)(par * V.par), pq = (unsigned)V.par - pp;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int nu = k < MU ? k : k + 1;
        const unsigned nu_p = (unsigned)(nu * V.dir) + pp, nu_q = (unsigned)(nu * V.dir) + pq;
        const unsigned mu_q = (unsigned)(MU * V.dir) + pq;
        v[k][0] = V.at(nu_q, s.p[MU]);
        v[k][1] = V.at(mu_q, s.p[nu]);
        v[k][2] = V.at(nu_p, s.c);
        v[k][3] = V.at(nu_q, s.m[nu]);
        v[k][4] = V.at(nu_p, s.p[MU] + (s.m[nu] - s.c));
        v[k][5] = V.at(mu_q, s.m[nu]);
    }
}

// One pass over the directions and parities, a work-item per link of a phase.
// (Keeping a work-item's offsets in registers from phase to phase measured no
// faster than reading its record again: 4^4 27.0 us a sweep either way, 8^3 x 4
// inside slabs 44.5 against 46.8.)
template <typename real, int KIND>
__device__ inline void slab_pass(const SlabView<real>& V, const SlabNb* nbr, HbQ<real>* wave_q, const SlabBlock& B,
                                 const EnsDesc& E, uint32_t ctr, double metro_delta)
{
    const int tid = (int)threadIdx.x;
#pragma unroll 1
    for (int phase = 0; phase < 8; ++phase) {
        const int mu = phase >> 1, par = phase & 1;
        // layers this direction updates: all of a lattice, or of a slab the
        // inner ones (spatial links) and all but the one above (temporal links)
        const int l0 = B.tau && mu < 3 ? 1 : 0;
        const int n = ((B.tau ? B.tau : B.nt) - l0) * B.slice;
        if ((tid & ~63) < n) {  // uniform for the wave
            const bool active = tid < n;
            const int lr = fdiv_small(active ? tid : 0, B.inv_slice);
            const int h = (active ? tid : 0) - lr * B.slice, l = lr + l0;
            const SlabNb w = nbr[h];
            const int odd = -((int)(w.par + (unsigned)(l + B.t0 + par)) & 1);  // all ones or none; x = 2 xh + (0 or 1)
            const unsigned base = (unsigned)(l * V.layer), self_h = (unsigned)(h * (int)sizeof(real));
            SlabSite s;
            s.c = base + self_h;
            s.p[0] = base + (odd ? w.x >> 16 : self_h), s.m[0] = base + (odd ? self_h : w.x & 0xFFFFu);
            s.p[1] = base + (w.y >> 16), s.m[1] = base + (w.y & 0xFFFFu);
            s.p[2] = base + (w.z >> 16), s.m[2] = base + (w.z & 0xFFFFu);
            // (inside a slab the layers above and below are there; a lattice wraps)
            s.p[3] = s.c + (unsigned)(l + 1 == B.layers ? V.layer - V.par : V.layer);
            s.m[3] = s.c + (unsigned)(l == 0 ? V.par - V.layer : -V.layer);
            real v[3][6];
            switch (mu) {
            case 0: gather_lds<real, 0>(V, s, par, v); break;
            case 1: gather_lds<real, 1>(V, s, par, v); break;
            case 2: gather_lds<real, 2>(V, s, par, v); break;
            default: gather_lds<real, 3>(V, s, par, v); break;
            }
            real& self = V.at((unsigned)(mu * V.dir + par * V.par), s.c);
            // canonical site 2 (h + slice t) + odd
            const int t = l + B.t0 < B.nt ? l + B.t0 : l + B.t0 - B.nt;
            const uint32_t lid = (uint32_t)mu + (uint32_t)(odd & 4) + 8u * ((uint32_t)h + (uint32_t)B.slice * (uint32_t)t);
            Block4 b0{};
            if (KIND != 1) b0 = philox4x32_10(lid, ctr, 0u, KIND == 2 ? DOM_METRO : DOM_HB, E.seed, E.key_id);
            const real th = update_link<real, KIND>(active, v, b0, lid, ctr, E.beta, E.seed, E.key_id, metro_delta,
                                                    wave_q, [&] { return self; });
            if (active) self = th;
        }
        __syncthreads();
    }
}

template <typename real, int STOCH>
__global__ void __launch_bounds__(kSlabThreads<real>)
    k_slab(const EnsDesc* __restrict__ ens, const SlabBlock* __restrict__ blocks, real* __restrict__ links,
           const uint32_t* __restrict__ upd, int pass_offset, int n_sweeps, int n_or, double metro_delta)
{
    extern __shared__ __align__(16) unsigned char slab_bytes[];
    const SlabBlock B = blocks[blockIdx.x];
    const EnsDesc& E = ens[B.e];
    const int tid = (int)threadIdx.x, T = (int)blockDim.x;
    SlabNb* nbr = reinterpret_cast<SlabNb*>(slab_bytes);
    HbQ<real>* queue = reinterpret_cast<HbQ<real>*>(nbr + B.slice);
    constexpr int w = sizeof(real);
    const int layer = B.slice * w, par_stride = B.layers * layer;
    const SlabView<real> V{reinterpret_cast<char*>(queue + (STOCH == 0 ? T : 0)), layer, par_stride, 2 * par_stride};

    const int sz = B.nxh * B.ny;
    for (int h = tid; h < B.slice; h += T) {
        const int yz = fdiv_small(h, B.inv_nxh), xh = h - yz * B.nxh;
        const int z = fdiv_small(yz, B.inv_ny), y = yz - z * B.ny;
        const int yp = y == B.ny - 1 ? h + B.nxh - sz : h + B.nxh, ym = y == 0 ? h + sz - B.nxh : h - B.nxh;
        const int zp = h + sz >= B.slice ? h + sz - B.slice : h + sz, zm = h < sz ? h + B.slice - sz : h - sz;
        const int xp = xh == B.nxh - 1 ? h + 1 - B.nxh : h + 1, xm = xh == 0 ? h + B.nxh - 1 : h - 1;
        nbr[h] = SlabNb{(unsigned)(yp * w) << 16 | (unsigned)(ym * w), (unsigned)(zp * w) << 16 | (unsigned)(zm * w),
                        (unsigned)(xp * w) << 16 | (unsigned)(xm * w), (unsigned)(y + z)};
    }
    // the layers of every (direction, parity) array, a slice each, in memory as in LDS
    auto copy = [&](bool in) {
        for (int a = 0; a < 8 * B.layers; ++a) {
            const int arr = a / B.layers, lay = a - arr * B.layers;
            // in: not the temporal links of the layer above a slab; out: not that layer, nor frozen links
            if (B.tau && lay == B.tau && (arr >= 6 || !in)) continue;
            if (B.tau && lay == 0 && arr < 6 && !in) continue;
            const int t = B.t0 + lay < B.nt ? B.t0 + lay : B.t0 + lay - B.nt;
            real* g = links + B.link_off + ((size_t)arr * B.vh + (size_t)t * B.slice);
            real* l = reinterpret_cast<real*>(V.lds + a * V.layer);
            if (in)
                for (int h = tid; h < B.slice; h += T) l[h] = g[h];
            else
                for (int h = tid; h < B.slice; h += T) g[h] = l[h];
        }
    };
    copy(true);
    __syncthreads();
    const uint32_t ctr = upd[B.e] + (uint32_t)pass_offset;
    HbQ<real>* wave_q = queue + (STOCH == 0 ? (tid & ~63) : 0);
    for (int k = 0; k < n_sweeps; ++k) {
        slab_pass<real, STOCH>(V, nbr, wave_q, B, E, ctr + (uint32_t)k, metro_delta);
#pragma unroll 1
        for (int j = 0; j < n_or; ++j) slab_pass<real, 1>(V, nbr, wave_q, B, E, 0u, metro_delta);
    }
    copy(false);
}

hipError_t launch_slab(const SlabLaunch& a)
{
    if (a.total_blocks <= 0 || a.n_sweeps <= 0) return hipSuccess;
    const int max_t = a.precision == 0 ? kSlabThreads<double> : kSlabThreads<float>;
    if (a.block < 64 || a.block > max_t || a.block % 64 || (a.stoch != 0 && a.stoch != 2)) return hipErrorInvalidValue;
    const dim3 g(a.total_blocks), b(a.block);
    if (a.precision == 0) {
        if (a.stoch == 0)
            hipLaunchKernelGGL((k_slab<double, 0>), g, b, a.lds_bytes, a.st, a.d_ens, a.d_blocks, (double*)a.links,
                               a.d_upd, a.pass_offset, a.n_sweeps, a.n_or, a.metro_delta);
        else
            hipLaunchKernelGGL((k_slab<double, 2>), g, b, a.lds_bytes, a.st, a.d_ens, a.d_blocks, (double*)a.links,
                               a.d_upd, a.pass_offset, a.n_sweeps, a.n_or, a.metro_delta);
    } else {
        if (a.stoch == 0)
            hipLaunchKernelGGL((k_slab<float, 0>), g, b, a.lds_bytes, a.st, a.d_ens, a.d_blocks, (float*)a.links,
                               a.d_upd, a.pass_offset, a.n_sweeps, a.n_or, a.metro_delta);
        else
            hipLaunchKernelGGL((k_slab<float, 2>), g, b, a.lds_bytes, a.st, a.d_ens, a.d_blocks, (float*)a.links,
                               a.d_upd, a.pass_offset, a.n_sweeps, a.n_or, a.metro_delta);
    }
    return hipGetLastError();
}

}  // namespace u1ml
