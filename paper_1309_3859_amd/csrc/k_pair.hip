// k_pair.hip -- both parities of one direction's checkerboard update in one
// launch.
//
// Paper: Amado, Cardoso, Bicudo, arXiv 1309.3859, Sec. II (local updates with
// 3 overrelaxation steps), Sec. II.C.1 and Algorithm 1 (frozen boundary
// spatial links), Sec. II.D (even then odd sites).
//
// The links of direction mu meet only across mu: link (x, mu) has link
// (x +- nu, mu), nu != mu, of the other parity in its staples, and no link of
// another position along mu.  A work-group owns a tile of rows (all of x at
// one (y, z, t)), the core, and updates first the even links of the core and
// of the rows one step around it (the halo), keeps them in LDS, then the odd
// links of the core from them.  An even halo link is updated by its own tile
// as well, from the same angles and the same Philox block, so both get the
// same bits.  Because neighbours still read a core's old angles, the new ones
// go to the other of two link buffers: every direction has a current buffer
// (byte offset src_d), and the launch turns mu's over to dst.  Rows whose
// neighbours are all in the tile (the whole extent, or frozen layers on both
// sides) have no halo.  All loads of both parities are issued before the
// first arithmetic.
//
// What bounds it: the launch (1.85 us with its loads and stores) and the
// instruction chain of the two updates; against two launches of one parity
// the launch is paid once.  The tile (host: pair_tile) is the one with the
// least work per SIMD, halo included.
#include "link_update.hpp"
#include "u1ml_internal.hpp"

namespace u1ml {

template <typename real, int KIND, int MU>
__global__ void __launch_bounds__(kPairThreads<real>)
    k_pair(const EnsDesc* __restrict__ ens, const PairBlock* __restrict__ blocks, const PairRow* __restrict__ rows,
           real* __restrict__ links, const uint32_t* __restrict__ upd, int pass_offset, unsigned src0, unsigned src1,
           unsigned src2, unsigned src3, unsigned dst, double metro_delta)
{
    constexpr int w = sizeof(real);
    __shared__ real even[kPairThreads<real>];
    __shared__ HbQ<real> queue[KIND == 0 ? kPairThreads<real> : 1];
    PairBlock B = blocks[blockIdx.x];
    asm volatile("" : "+s"(B.base), "+s"(B.n1), "+s"(B.row_tab), "+s"(B.nxh), "+s"(B.inv_nxh), "+s"(B.link_off));
    const EnsDesc& E = ens[B.e];
    const int tid = (int)threadIdx.x;
    if ((tid & ~63) >= B.n1) return;  // no link in this wave (ended waves do not count at the barrier)
    const bool first = tid < B.n1, second = tid < B.n2;
    const int item = first ? tid : 0;
    const int row = fdiv_small(item, B.inv_nxh);
    const int xh = item - __mul24(row, B.nxh);
    const PairRow R = rows[B.row_tab + row];
    // x of the row's even site is 2 xh + odd, of its odd site 2 xh + 1 - odd
    const int odd = -((R.par + B.par) & 1);  // all ones or none
    const int xb = xh * w, sy = B.nxh * w, o = xb + B.base;
    const int xp = xh == B.nxh - 1 ? w - sy : w, xm = xh == 0 ? sy - w : -w;
    SiteNb nb;
    nb.c = (unsigned)(R.c + o);
    nb.p[1] = (unsigned)(R.p1 + o), nb.m[1] = (unsigned)(R.m1 + o);
    nb.p[2] = (unsigned)(R.p2 + o), nb.m[2] = (unsigned)(R.m2 + o);
    nb.p[3] = (unsigned)(R.p3 + o), nb.m[3] = (unsigned)(R.m3 + o);
    nb.p[0] = nb.c + (unsigned)(xp & odd);
    nb.m[0] = nb.c + (unsigned)(xm & ~odd);
    SiteNb nc = nb;  // the odd site of the same half index
    nc.p[0] = nb.c + (unsigned)(xp & ~odd);
    nc.m[0] = nb.c + (unsigned)(xm & odd);

    const LinkBuf<real> lb(links + B.link_off);
    const unsigned vhb = (unsigned)B.vh * w;
    const unsigned src[4] = {src0, src1, src2, src3};
    const unsigned self = MU * 2 * vhb;  // the even links; the odd ones follow at + vhb
    real v1[3][6], v2[3][6], old1 = real(0), old2 = real(0), fp = real(0), fm = real(0);
    gather_nb<real, MU, Nu<MU, 0>::v, false>(lb, vhb, src, nb, 0, v1[0]);
    gather_nb<real, MU, Nu<MU, 1>::v, false>(lb, vhb, src, nb, 0, v1[1]);
    gather_nb<real, MU, Nu<MU, 2>::v, false>(lb, vhb, src, nb, 0, v1[2]);
    if (KIND != 0) old1 = lb.ld(nb.c, self + src[MU]);
    // (halo lanes load these as well and leave them unused: no branch between the loads)
    gather_nb<real, MU, Nu<MU, 0>::v, true>(lb, vhb, src, nc, 1, v2[0]);
    gather_nb<real, MU, Nu<MU, 1>::v, true>(lb, vhb, src, nc, 1, v2[1]);
    gather_nb<real, MU, Nu<MU, 2>::v, true>(lb, vhb, src, nc, 1, v2[2]);
    if (KIND != 0) old2 = lb.ld(nc.c, self + vhb + src[MU]);
    if (MU < 3) {  // the even links one step in t, where they are frozen
        fp = lb.ld(nc.p[3], self + src[MU]);
        fm = lb.ld(nc.m[3], self + src[MU]);
    }
    // Philox: canonical site 2 h + (0 or 1), h the half index
    const uint32_t ctr = KIND == 1 ? 0u : upd[B.e] + (uint32_t)pass_offset;
    const uint32_t lid1 = (uint32_t)MU + nb.c * (8u / w) + (uint32_t)(4 & odd);
    Block4 b1{}, b2{};
    if (KIND != 1) {
        b1 = philox4x32_10(lid1, ctr, 0u, KIND == 2 ? DOM_METRO : DOM_HB, E.seed, E.key_id);
        b2 = philox4x32_10(lid1 ^ 4u, ctr, 0u, KIND == 2 ? DOM_METRO : DOM_HB, E.seed, E.key_id);
    }
    HbQ<real>* wave_q = queue + (KIND == 0 ? (tid & ~63) : 0);

    auto update = [&](bool active, const real (&v)[3][6], const Block4& b, uint32_t lid, real old, unsigned self_off) {
        return update_link<real, KIND>(active, v, b, lid, ctr, E.beta, E.seed, E.key_id, metro_delta, wave_q,
                                       [&] { return KIND == 0 ? lb.ld(nb.c, self_off + src[MU]) : old; });
    };
    // the even links one step across mu, from LDS
    auto across = [&] {
        auto lds = [&](unsigned code, real frozen) {
            return code == kPairFrozen ? frozen
                                       : *reinterpret_cast<const real*>(reinterpret_cast<const char*>(even) + code + xb);
        };
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int nu = k < MU ? k : k + 1;
            const unsigned code = nu == 1 ? R.ly : (nu == 2 ? R.lz : R.lt);
            const char* me = reinterpret_cast<const char*>(even) + item * w;
            v2[k][1] = nu == 0 ? *reinterpret_cast<const real*>(me + (xp & ~odd)) : lds(code >> 16, fp);
            v2[k][5] = nu == 0 ? *reinterpret_cast<const real*>(me + (xm & odd)) : lds(code & 0xFFFFu, fm);
        }
    };
    if constexpr (KIND == 1 && sizeof(real) == 4) {
        const real th1 = update(first, v1, b1, lid1, old1, self);
        even[tid] = th1;
        if (second) lb.st(th1, nb.c, self + dst);
        __syncthreads();
        if (second) {
            across();
            lb.st(update(true, v2, b2, lid1, old2, self + vhb), nb.c, self + vhb + dst);
        }
    } else {
        // both parities through the same code: straight-line code costs about
        // 1.3 ns an instruction to fetch, so the long updates are a loop
        int two = 2;
        asm volatile("" : "+s"(two));  // (keeps the compiler from unrolling it)
#pragma unroll 1
        for (int ph = 0, n = two; ph < n; ++ph) {
            const real th = update(ph == 0 ? first : second, v1, b1, ph == 0 ? lid1 : lid1 ^ 4u, old1, self + (unsigned)ph * vhb);
            if (second) lb.st(th, nb.c, self + (unsigned)ph * vhb + dst);
            if (ph != 0) break;
            even[tid] = th;
            __syncthreads();
            if ((tid & ~63) >= B.n2) break;
            across();
#pragma unroll
            for (int k = 0; k < 18; ++k) v1[k / 6][k % 6] = v2[k / 6][k % 6];
            b1 = b2;
            old1 = old2;
        }
    }
}

template <typename real, int KIND>
static void launch_pair_t(const PairLaunch& a)
{
    const dim3 g(a.total_blocks), b(a.block);
    real* lk = (real*)a.links;
    switch (a.mu) {
    case 0: hipLaunchKernelGGL((k_pair<real, KIND, 0>), g, b, 0, a.st, a.d_ens, a.d_blocks, a.d_rows, lk, a.d_upd, a.pass_offset, a.src[0], a.src[1], a.src[2], a.src[3], a.dst, a.metro_delta); break;
    case 1: hipLaunchKernelGGL((k_pair<real, KIND, 1>), g, b, 0, a.st, a.d_ens, a.d_blocks, a.d_rows, lk, a.d_upd, a.pass_offset, a.src[0], a.src[1], a.src[2], a.src[3], a.dst, a.metro_delta); break;
    case 2: hipLaunchKernelGGL((k_pair<real, KIND, 2>), g, b, 0, a.st, a.d_ens, a.d_blocks, a.d_rows, lk, a.d_upd, a.pass_offset, a.src[0], a.src[1], a.src[2], a.src[3], a.dst, a.metro_delta); break;
    default: hipLaunchKernelGGL((k_pair<real, KIND, 3>), g, b, 0, a.st, a.d_ens, a.d_blocks, a.d_rows, lk, a.d_upd, a.pass_offset, a.src[0], a.src[1], a.src[2], a.src[3], a.dst, a.metro_delta); break;
    }
}

hipError_t launch_pair(const PairLaunch& a)
{
    if (a.total_blocks <= 0) return hipSuccess;
    if (a.kind < 0 || a.kind > 2 || a.mu < 0 || a.mu > 3) return hipErrorInvalidValue;
    if (a.block < 64 || a.block > (a.precision == 0 ? kPairThreads<double> : kPairThreads<float>) || a.block % 64)
        return hipErrorInvalidValue;
    if (a.precision == 0) {
        if (a.kind == 0) launch_pair_t<double, 0>(a);
        else if (a.kind == 1) launch_pair_t<double, 1>(a);
        else launch_pair_t<double, 2>(a);
    } else {
        if (a.kind == 0) launch_pair_t<float, 0>(a);
        else if (a.kind == 1) launch_pair_t<float, 1>(a);
        else launch_pair_t<float, 2>(a);
    }
    return hipGetLastError();
}

// The other link buffer's copy of the lane's links (so that frozen links,
// which no update writes, are in both): `bytes` of every ensemble at its
// offset, to the same offset `alt` bytes further.
template <typename real>
__global__ void __launch_bounds__(256) k_mirror(const EnsDesc* __restrict__ ens, real* __restrict__ links, unsigned alt)
{
    const EnsDesc& E = ens[blockIdx.y];
    const size_t n16 = (size_t)8 * E.vh * sizeof(real) / 16;  // 4 V words, V a multiple of 16
    const uint4* src = reinterpret_cast<const uint4*>(links + E.link_off);
    uint4* dst = reinterpret_cast<uint4*>(reinterpret_cast<char*>(links + E.link_off) + alt);
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += (size_t)gridDim.x * 256) dst[i] = src[i];
}

hipError_t launch_mirror(const EnsDesc* d_ens, int n_ens, int precision, void* links, unsigned alt, int blocks,
                         hipStream_t st)
{
    if (n_ens <= 0) return hipSuccess;
    const dim3 g(blocks, n_ens);
    if (precision == 0)
        hipLaunchKernelGGL(k_mirror<double>, g, dim3(256), 0, st, d_ens, (double*)links, alt);
    else
        hipLaunchKernelGGL(k_mirror<float>, g, dim3(256), 0, st, d_ens, (float*)links, alt);
    return hipGetLastError();
}

}  // namespace u1ml
