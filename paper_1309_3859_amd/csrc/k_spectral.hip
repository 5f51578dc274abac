// k_spectral.hip -- the insertion estimators in spectral form.
//
// Paper: Amado, Cardoso, Bicudo, arXiv 1309.3859, Sec. II.C.3 (insertion
// estimator <P^dagger P O> = 1/(N_sigma N_t |M|) sum_x sum_mu sum_S [TO](S)
// prod_{S' != S} [T](S'), [TO] the slab average of T^(tau) times the slab
// sum of O at the probe site) and Sec. II.C.2 (two levels: T^(4), TO^(4)).
//
// Written out over the stored measurements m of every inner level k, with
// thin slab s inside thick slab S (one level: a single thick slab of all the
// slabs, and W = 1):
//   sum_x sum_S [TO](S) W_S = 1/(n_o n_i) sum_k sum_s sum_m sum_x G_k(x,s) T_m(x,s) O_m(x + d, s),
//   G_k(x, s) = W_S(x) prod_{s' in S, s' != s} [T]_k(x, s'),   W_S = prod_{S' != S} A(S'),
// A the outer averages.  For a charge axis, a slab, a separation and a
// component, the sum over x for every transverse displacement p = (p1, p2)
// at once is a cross-correlation over the plane orthogonal to the axis.  With
// the plane transform X^(k) = sum_{u,v} X(u,v) exp(-2 pi i (k1 u/n1 + k2 v/n2))
// and h^~ the transform with the conjugate kernel:
//   sum_x h(x) O(x + l e_par + p)
//     = 1/(n1 n2) sum_k exp(+2 pi i (k1 p1/n1 + k2 p2/n2)) sum_{x_par} O^_{x_par + l}(k) h^~_{x_par}(k).
// The inner sum is accumulated over measurements and inner levels per
// (axis, slab, r, component, kind, probe group); the probes' displacements
// are read off once per configuration.  Memory is independent of the number
// of probes.
#include <algorithm>

#include "device_common.hpp"
#include "scaled.hpp"
#include "u1ml_internal.hpp"

namespace u1ml {

namespace {

__device__ inline int find_ens_s(const int* __restrict__ bstart, int n_ens, int bid)
{
    int e = 0;
    for (int end = n_ens; end - e > 1;) {
        const int mid = (e + end) >> 1;
        if (bid >= bstart[mid])
            e = mid;
        else
            end = mid;
    }
    return e;
}

__device__ inline double2 cmul(double2 a, double2 b) { return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }

__device__ inline int orient_of(int c, int dir) { return c < 3 ? (dir + c) % 3 : 3 + (dir + c - 3) % 3; }
__device__ inline int extent(const EnsDesc& E, int dir) { return dir == 0 ? E.nx : dir == 1 ? E.ny : E.nz; }
__device__ inline bool spans_axis(int c) { return c == 0 || c == 4 || c == 5; }

// Position of site xs = x + nx (y + ny z) in the plane-major order of charge
// axis dir: (x_par n1 + u) n2 + v, with (x_par, u, v) the coordinates along
// (dir, d1, d2), d1 = dir + 1 and d2 = dir + 2 (mod 3); each plane x_par is
// then one contiguous run of n1 n2 sites.
__device__ inline int plane_index(int xs, int dir, int nx, int ny, int nz)
{
    const int x = xs % nx, yz = xs / nx;
    const int y = yz % ny, z = yz / ny;
    const int xp = dir == 0 ? x : dir == 1 ? y : z;
    const int u = dir == 0 ? y : dir == 1 ? z : x;
    const int v = dir == 0 ? z : dir == 1 ? x : y;
    const int n1 = dir == 0 ? ny : dir == 1 ? nz : nx;
    const int n2 = dir == 0 ? nz : dir == 1 ? nx : ny;
    return (xp * n1 + u) * n2 + v;
}

struct dds {
    double hi, lo;
};

__device__ inline dds dds_add(dds a, double b)
{
    const double s = a.hi + b;
    const double bb = s - a.hi;
    const double err = (a.hi - (s - bb)) + (b - bb) + a.lo;
    const double hi = s + err;
    return dds{hi, err - (hi - s)};
}

}  // namespace

// ---------------------------------------------------------------------------
// Weights.  One work-item per (ensemble, axis, r, x); it writes every slab.
//   k_wfac: W[axis, r][S][x] = 2^-E(r) prod_{S' != S} scale * out_t[axis, r][S'][x]
//   k_gfac: G[axis, r][s][x] = W_S(x) prod_{s' in S, s' != s} avg_t[axis, r][s'][x]
//           (q thin slabs per thick slab, q = 0 for all slabs; W = 2^-E(r) when
//           wf is null), stored in the plane-major order of the axis (plane_index)
// E(r) is the exponent of the configuration's correlator products, read from
// its record, so that the spectral sums come out relative to the same 2^E(r)
// as the correlator.  The products over slabs run as scaled complex numbers,
// over ascending slab index.
// ---------------------------------------------------------------------------
__device__ inline int record_exp(const EnsDesc& E, const ObsDesc& O, const double* __restrict__ results,
                                 const int* __restrict__ ring, int ir)
{
    const double* rec = results + ((size_t)(*ring) * O.n_ens_total + E.res_index) * O.n_doubles_per_config;
    return (int)rec[O.n_doubles_per_config - O.n_r + ir];
}

__global__ void __launch_bounds__(256) k_wfac(const EnsDesc* __restrict__ ens, const int* __restrict__ bstart,
                                              int n_ens, const ObsDesc* __restrict__ obs,
                                              const double2* __restrict__ out_t, double scale,
                                              double2* __restrict__ wf, const double* __restrict__ results,
                                              const int* __restrict__ ring)
{
    const int e = find_ens_s(bstart, n_ens, blockIdx.x);
    const EnsDesc& E = ens[e];
    const long long item = (long long)(blockIdx.x - bstart[e]) * blockDim.x + threadIdx.x;
    const int nsig = E.nsig, So = E.s_out;
    if (item >= (long long)obs->n_dirs * obs->n_r * nsig) return;
    const int xs = (int)(item % nsig);
    const long long idr = item / nsig;
    const int Er = record_exp(E, *obs, results, ring, (int)(idr % obs->n_r));
    for (int S = 0; S < So; ++S) {
        sc w{1.0, 0.0, 0};
        for (int S2 = 0; S2 < So; ++S2) {
            if (S2 == S) continue;
            double2 a = out_t[E.ot_off + ((size_t)idr * So + S2) * nsig + xs];
            a.x *= scale;
            a.y *= scale;
            w = sc_mul(w, a);
        }
        wf[E.wf_off + ((size_t)idr * So + S) * nsig + xs] = sc_rel(w, Er);
    }
}

__global__ void __launch_bounds__(256) k_gfac(const EnsDesc* __restrict__ ens, const int* __restrict__ bstart,
                                              int n_ens, const ObsDesc* __restrict__ obs,
                                              const double2* __restrict__ avg_t, const double2* __restrict__ wf,
                                              int q, double2* __restrict__ gf, const double* __restrict__ results,
                                              const int* __restrict__ ring)
{
    const int e = find_ens_s(bstart, n_ens, blockIdx.x);
    const EnsDesc& E = ens[e];
    const long long item = (long long)(blockIdx.x - bstart[e]) * blockDim.x + threadIdx.x;
    const int nsig = E.nsig, Si = E.s_in, So = E.s_out;
    if (item >= (long long)obs->n_dirs * obs->n_r * nsig) return;
    const int xs = (int)(item % nsig);
    const long long idr = item / nsig;
    const int qq = q > 0 ? q : Si;  // q = 0: one thick slab of every slab (one level)
    const int pidx = plane_index(xs, obs->dirs[idr / obs->n_r], E.nx, E.ny, E.nz);
    const int Er = wf ? 0 : record_exp(E, *obs, results, ring, (int)(idr % obs->n_r));
    for (int s = 0; s < Si; ++s) {
        const int S = s / qq;
        sc g{1.0, 0.0, 0};
        if (wf) {
            const double2 w = wf[E.wf_off + ((size_t)idr * So + S) * nsig + xs];
            g = sc{w.x, w.y, 0};
        }
        for (int s2 = S * qq; s2 < S * qq + qq; ++s2) {
            if (s2 == s) continue;
            g = sc_mul(g, avg_t[E.at_off + ((size_t)idr * Si + s2) * nsig + xs]);
        }
        gf[E.gf_off + ((size_t)idr * Si + s) * nsig + pidx] = sc_rel(g, Er);
    }
}

// One axis of the plane transform, in LDS:
//   out[a oa + b ob] = sum_c in[a sa + c sc] tw[(b c) mod nc],  a < na, b < nc,
// every thread owning a TxT tile of (a, b) so that each loaded input and
// twiddle serves T products.  na and nc are multiples of T.
template <int T>
__device__ inline void dft_axis(const double2* __restrict__ in, int na, int nc, int sa, int sc,
                                const double2* __restrict__ tw, double2* __restrict__ out, int oa, int ob)
{
    const int nbt = nc / T;
    const int tiles = (na / T) * nbt;
    for (int t = threadIdx.x; t < tiles; t += blockDim.x) {
        const int a0 = (t / nbt) * T, b0 = (t - (t / nbt) * nbt) * T;
        double re[T][T], im[T][T];
        int ph[T];
#pragma unroll
        for (int j = 0; j < T; ++j) {
            ph[j] = 0;
#pragma unroll
            for (int i = 0; i < T; ++i) re[i][j] = im[i][j] = 0.0;
        }
        for (int c = 0; c < nc; ++c) {
            double2 x[T], w[T];
#pragma unroll
            for (int i = 0; i < T; ++i) x[i] = in[(a0 + i) * sa + c * sc];
#pragma unroll
            for (int j = 0; j < T; ++j) {
                w[j] = tw[ph[j]];
                ph[j] += b0 + j;
                if (ph[j] >= nc) ph[j] -= nc;
            }
#pragma unroll
            for (int i = 0; i < T; ++i)
#pragma unroll
                for (int j = 0; j < T; ++j) {
                    re[i][j] += x[i].x * w[j].x - x[i].y * w[j].y;
                    im[i][j] += x[i].x * w[j].y + x[i].y * w[j].x;
                }
        }
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
            for (int j = 0; j < T; ++j) out[(a0 + i) * oa + (b0 + j) * ob] = make_double2(re[i][j], im[i][j]);
    }
}

// ---------------------------------------------------------------------------
// Mixed-radix FFT along one axis of a plane in LDS (Stockham autosort, radices
// 4, 2, 3, 5 in that order; Cooley & Tukey 1965, Stockham 1966).  Stage with
// radix R after the radices so far have product Ns: butterfly j of a sequence
// of length n takes the R inputs j + r n/R, multiplies input r by
// w^(r (j mod Ns) n/(Ns R)), forms their length-R transform and writes output
// q to (j div Ns) Ns R + (j mod Ns) + q Ns; after the last stage the sequence
// holds its transform in natural order.  w = exp(sg 2 pi i / n) comes from the
// table tw (n entries), so the forward and the conjugate kernel share the
// code.  Results differ from the direct sum only by rounding, and are the same
// for every launch shape.
// ---------------------------------------------------------------------------
struct FftPlan {
    int c4, c2, c3, c5;  // stages of each radix, applied in this order
    int n_st;            // total, 0 if n has a prime factor above 5
};

__device__ inline FftPlan fft_plan(int n)
{
    FftPlan p{0, 0, 0, 0, 0};
    while (n % 4 == 0) { ++p.c4; n /= 4; }
    while (n % 2 == 0) { ++p.c2; n /= 2; }
    while (n % 3 == 0) { ++p.c3; n /= 3; }
    while (n % 5 == 0) { ++p.c5; n /= 5; }
    p.n_st = n == 1 ? p.c4 + p.c2 + p.c3 + p.c5 : 0;
    return p;
}

// One stage over `rows` sequences: element i of sequence q at src[q sq + i se],
// written to dst[q dq + i de].  Consecutive work-items take consecutive
// butterflies of one sequence when the elements of a sequence are adjacent
// (se = 1), else the same butterfly of consecutive sequences (sq = 1), so the
// 16-byte LDS accesses of a wave stay on distinct banks and the last stage's
// global stores are contiguous.
template <int R>
__device__ inline void fft_stage(const double2* __restrict__ src, int sq, int se, double2* __restrict__ dst, int dq,
                                 int de, int n, int rows, int Ns, const double2* __restrict__ tw, double sg)
{
    const int m = n / R;
    const int tstep = n / (Ns * R);
    const int total = rows * m;
    const bool qfast = se != 1;
    for (int b = threadIdx.x; b < total; b += blockDim.x) {
        const int q = qfast ? b % rows : b / m;
        const int j = qfast ? b / rows : b - q * m;
        const int k = j % Ns;
        double2 v[R];
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = src[q * sq + (j + r * m) * se];
#pragma unroll
        for (int r = 1; r < R; ++r) v[r] = cmul(v[r], tw[r * k * tstep]);  // r k tstep < n
        double2 V[R];
        if (R == 2) {
            V[0] = make_double2(v[0].x + v[1].x, v[0].y + v[1].y);
            V[1] = make_double2(v[0].x - v[1].x, v[0].y - v[1].y);
        } else if (R == 4) {
            // w_4 = sg i: w z = sg (-z.y, z.x)
            const double2 a = make_double2(v[0].x + v[2].x, v[0].y + v[2].y);
            const double2 c = make_double2(v[0].x - v[2].x, v[0].y - v[2].y);
            const double2 bb = make_double2(v[1].x + v[3].x, v[1].y + v[3].y);
            const double2 d = make_double2(v[1].x - v[3].x, v[1].y - v[3].y);
            const double2 wd = make_double2(-sg * d.y, sg * d.x);
            V[0] = make_double2(a.x + bb.x, a.y + bb.y);
            V[1] = make_double2(c.x + wd.x, c.y + wd.y);
            V[2] = make_double2(a.x - bb.x, a.y - bb.y);
            V[3] = make_double2(c.x - wd.x, c.y - wd.y);
        } else {
            const int nr = n / R;
#pragma unroll
            for (int qq = 0; qq < R; ++qq) {
                double2 acc = v[0];
#pragma unroll
                for (int r = 1; r < R; ++r) {
                    const double2 w = tw[((r * qq) % R) * nr];
                    acc.x += v[r].x * w.x - v[r].y * w.y;
                    acc.y += v[r].x * w.y + v[r].y * w.x;
                }
                V[qq] = acc;
            }
        }
        const int idx = (j / Ns) * Ns * R + k;
#pragma unroll
        for (int qq = 0; qq < R; ++qq) dst[q * dq + (idx + qq * Ns) * de] = V[qq];
    }
}

// The whole FFT along one axis: input in LDS buffer `cur` (sequence stride sq,
// element stride se), stages ping-pong between `cur` and `other` (same
// strides), the last stage writes to out[q oq + k oe] (global memory, or the
// LDS buffer that the last stage does not read).
__device__ inline void fft_axis(const FftPlan& P, double2* cur, double2* other, int sq, int se, int n, int rows,
                                const double2* tw, double sg, double2* out, int oq, int oe)
{
    int Ns = 1;
    for (int st = 0; st < P.n_st; ++st) {
        const bool last = st == P.n_st - 1;
        double2* dst = last ? out : other;
        const int dq = last ? oq : sq, de = last ? oe : se;
        const int R = st < P.c4 ? 4 : st < P.c4 + P.c2 ? 2 : st < P.c4 + P.c2 + P.c3 ? 3 : 5;
        switch (R) {
        case 4: fft_stage<4>(cur, sq, se, dst, dq, de, n, rows, Ns, tw, sg); break;
        case 2: fft_stage<2>(cur, sq, se, dst, dq, de, n, rows, Ns, tw, sg); break;
        case 3: fft_stage<3>(cur, sq, se, dst, dq, de, n, rows, Ns, tw, sg); break;
        default: fft_stage<5>(cur, sq, se, dst, dq, de, n, rows, Ns, tw, sg); break;
        }
        __syncthreads();
        Ns *= R;
        double2* t = cur;
        cur = other;
        other = t;
    }
}

// ---------------------------------------------------------------------------
// Staging of measurement m_in for the plane transforms: the slab phases and
// the 12 O rows copied to the plane-major order of each charge axis, so that
// every plane the transforms read is contiguous.
//   cpl[axis][s][plane_index],  opl[axis][s][row][plane_index]
// Work-group per (ensemble, axis, slab, tile): the target's fastest
// coordinate is v (z for the x axis, x for the y axis, y for the z axis); a
// tile is 16 x values by 16 v values at fixed remaining coordinate, one per
// work-item, read with x fastest and written with v fastest through LDS, so
// both sides are contiguous.  For the y axis (v = x) the tile is 16 x values
// of 16 rows, copied directly.
// Bound by latency (48^3 x 12: 83 MB): tiles of 32 x 32 in three passes of
// four rows took 37 us, the passes as work-groups of their own 31 us, and
// half of the work-items of every second tile lie outside 48 sites; now 22 us (3.7 TB/s).
// ---------------------------------------------------------------------------
template <typename ot>
__global__ void __launch_bounds__(kStageTile * kStageTile) k_plane_stage(const EnsDesc* __restrict__ ens, const int* __restrict__ bstart,
                                                     int n_ens, const ObsDesc* __restrict__ obs,
                                                     const double2* __restrict__ hist_c, const ot* __restrict__ hist_o,
                                                     int m_in, double2* __restrict__ cpl, ot* __restrict__ opl)
{
    constexpr int TT = kStageTile;
    __shared__ double2 tc[TT][TT + 1];
    __shared__ ot to[12][TT][TT + 1];
    const int e = find_ens_s(bstart, n_ens, blockIdx.x);
    const EnsDesc& E = ens[e];
    const ObsDesc& O = *obs;
    const int nx = E.nx, ny = E.ny, nz = E.nz, nsig = E.nsig, Si = E.s_in;
    const int npm = max(nx, max(ny, nz));
    const int tx_n = (nx + TT - 1) / TT, tv_n = (npm + TT - 1) / TT;
    const int tiles = tx_n * tv_n * npm;  // per (axis, slab), sized for the largest extent
    int local = blockIdx.x - bstart[e];
    const int tile = local % tiles;
    local /= tiles;
    const int s = local % Si;
    const int id = local / Si;
    if (id >= O.n_dirs) return;
    const int dir = O.dirs[id];
    // v: the target's fastest axis; w: the remaining one (y axis: v = x, rows y, w = z)
    const int vax = dir == 0 ? 2 : dir == 1 ? 0 : 1;
    const int wax = dir == 0 ? 1 : 2;
    const int nrow = vax == 2 ? nz : ny;  // extent of the tile's second index
    const int x0 = (tile % tx_n) * TT;
    const int v0 = ((tile / tx_n) % tv_n) * TT;
    const int w = tile / (tx_n * tv_n);
    if (w >= extent(E, wax) || v0 >= nrow) return;  // uniform for the block
    const size_t ps = (size_t)id * Si + s;
    const double2* hc = hist_c + E.hc_off + ((size_t)m_in * Si + s) * nsig;
    const ot* ho = hist_o + E.ho_off + ((size_t)m_in * Si + s) * 12 * nsig;
    double2* dc = cpl + E.cpl_off + ps * nsig;
    ot* dob = opl + E.opl_off + ps * 12 * nsig;
    const int lx = threadIdx.x % TT, ly = threadIdx.x / TT;
    // read with x fastest, every load issued before the first store
    const int v = min(v0 + ly, nrow - 1), x = min(x0 + lx, nx - 1);
    const int y = vax == 2 ? w : v, z = vax == 2 ? v : w;
    const int xs = x + nx * (y + ny * z);
    const double2 c = hc[xs];
    ot o[12];
#pragma unroll
    for (int row = 0; row < 12; ++row) o[row] = ho[(size_t)row * nsig + xs];
    if (vax == 0) {
        // y axis: plane index (y nz + z) nx + x keeps x fastest: a plain copy of TT rows
        if (v0 + ly >= ny || x0 + lx >= nx) return;
        const int p = (y * nz + z) * nx + x;
        dc[p] = c;
#pragma unroll
        for (int row = 0; row < 12; ++row) dob[(size_t)row * nsig + p] = o[row];
        return;
    }
    tc[ly][lx] = c;
#pragma unroll
    for (int row = 0; row < 12; ++row) to[row][ly][lx] = o[row];
    __syncthreads();
    // write with v fastest: x axis p = (x ny + y) nz + z (y = w, z = v); z axis p = (z nx + x) ny + y (z = w, y = v)
    const int xw = x0 + ly, vw = v0 + lx;
    if (vw >= nrow || xw >= nx) return;
    const int p = vax == 2 ? (xw * ny + w) * nz + vw : (w * nx + xw) * ny + vw;
    dc[p] = tc[lx][ly];
#pragma unroll
    for (int row = 0; row < 12; ++row) dob[(size_t)row * nsig + p] = to[row][lx][ly];
}

// ---------------------------------------------------------------------------
// Plane transforms of measurement m_in.  Work-group per (ensemble, axis,
// slab s, field f, axis coordinate x_par); fields f < n_r are
// h = G(x,s,r) conj(c_m(x)) c_m(x + r e_par) (conjugate kernel), fields
// n_r .. n_r + 11 the O rows (orientation, kind) (plain kernel).  The plane
// is staged in LDS, transformed along v, then along u, by the mixed-radix
// FFT when both extents factor into 2, 3 and 5, else by direct sums over the
// axis in ascending order; twiddles exp(2 pi i j / n) come from sincospi in
// FP64.  Either way the outputs are the same for every launch shape.
//   sph[axis][s][r][x_par][k],  spo[axis][s][row][x_par][k],  k = k1 n2 + k2
// ---------------------------------------------------------------------------
constexpr int kPlaneThreads = 512;  // two work-groups fill a CU's LDS; more threads per plane hide latency

template <typename ot, int T>
__global__ void __launch_bounds__(kPlaneThreads) k_dft_planes(const EnsDesc* __restrict__ ens, const int* __restrict__ bstart,
                                                    int n_ens, const ObsDesc* __restrict__ obs,
                                                    const int* __restrict__ rlist, const double2* __restrict__ cpl,
                                                    const ot* __restrict__ opl, const double2* __restrict__ gf,
                                                    double2* __restrict__ sph, double2* __restrict__ spo)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int e = find_ens_s(bstart, n_ens, blockIdx.x);
    const EnsDesc& E = ens[e];
    const ObsDesc& O = *obs;
    const int nsig = E.nsig, Si = E.s_in, R = O.n_r, NF = R + 12;
    const int n3[3] = {E.nx, E.ny, E.nz};
    const int npm = max(E.nx, max(E.ny, E.nz));
    int local = blockIdx.x - bstart[e];
    const int xpar = local % npm;
    local /= npm;
    const int f = local % NF;
    local /= NF;
    const int s = local % Si;
    const int id = local / Si;
    if (id >= O.n_dirs) return;
    const int dir = O.dirs[id];
    const int N = n3[dir];
    if (xpar >= N) return;  // uniform for the block
    const int d1 = dir == 2 ? 0 : dir + 1, d2 = dir == 0 ? 2 : dir - 1;
    const int n1 = n3[d1], n2 = n3[d2], n12 = n1 * n2;
    double2* X = reinterpret_cast<double2*>(lds_raw);
    double2* Y = X + n12;
    double2* w1 = Y + n12;
    double2* w2 = w1 + n1;
    const double sg = f < R ? 1.0 : -1.0;  // sign of the kernel's exponent
    for (int j = threadIdx.x; j < n1; j += blockDim.x) {
        double sn, cs;
        sincospi(2.0 * (double)j / (double)n1, &sn, &cs);
        w1[j] = make_double2(cs, sg * sn);
    }
    for (int j = threadIdx.x; j < n2; j += blockDim.x) {
        double sn, cs;
        sincospi(2.0 * (double)j / (double)n2, &sn, &cs);
        w2[j] = make_double2(cs, sg * sn);
    }
    // the staged measurement and G are in plane-major order: plane x_par is
    // the contiguous run [x_par n12, (x_par + 1) n12)
    const size_t ps = (size_t)id * Si + s;
    if (f < R) {
        const int r = rlist[f];
        const double2* ca = cpl + E.cpl_off + ps * nsig + (size_t)xpar * n12;
        const double2* cb = cpl + E.cpl_off + ps * nsig + (size_t)((xpar + r) % N) * n12;
        const double2* g = gf + E.gf_off + (((size_t)id * R + f) * Si + s) * nsig + (size_t)xpar * n12;
        // four elements per work-item and round, all loads issued before any use
        for (int j0 = threadIdx.x; j0 < n12; j0 += 4 * blockDim.x) {
            double2 a[4], b[4], gg[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int j = min(j0 + u * (int)blockDim.x, n12 - 1);
                a[u] = ca[j];
                b[u] = cb[j];
                gg[u] = g[j];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int j = j0 + u * (int)blockDim.x;
                const double2 t = make_double2(a[u].x * b[u].x + a[u].y * b[u].y, a[u].x * b[u].y - a[u].y * b[u].x);
                if (j < n12) X[j] = cmul(gg[u], t);
            }
        }
    } else {
        const ot* op = opl + E.opl_off + (ps * 12 + (f - R)) * nsig + (size_t)xpar * n12;
        for (int j0 = threadIdx.x; j0 < n12; j0 += 4 * blockDim.x) {
            ot v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = op[min(j0 + u * (int)blockDim.x, n12 - 1)];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (j0 + u * (int)blockDim.x < n12) X[j0 + u * blockDim.x] = make_double2((double)v[u], 0.0);
        }
    }
    __syncthreads();
    double2* out = f < R ? sph + E.sph_off + (((size_t)id * Si + s) * R + f) * nsig + (size_t)xpar * n12
                         : spo + E.spo_off + (((size_t)id * Si + s) * 12 + (f - R)) * nsig + (size_t)xpar * n12;
    const FftPlan P1 = fft_plan(n1), P2 = fft_plan(n2);
    if (P1.n_st > 0 && P2.n_st > 0) {
        // along v (sequences u, contiguous), result left in X or Y, then along u
        // (sequences k2, stride n2), the last stage writing out[k1 n2 + k2]
        double2* mid = (P2.n_st & 1) ? Y : X;
        fft_axis(P2, X, Y, n2, 1, n2, n1, w2, sg, mid, n2, 1);
        fft_axis(P1, mid, mid == X ? Y : X, 1, n2, n1, n2, w1, sg, out, 1, n2);
        return;
    }
    // an extent with a prime factor above 5: direct sums (tiles of T x T outputs per thread)
    dft_axis<T>(X, n1, n2, n2, 1, w2, Y, n2, 1);
    __syncthreads();
    dft_axis<T>(Y, n2, n1, 1, n2, w1, out, 1, n2);
}

// ---------------------------------------------------------------------------
// Small DFTs in registers, kernel exp(+2 pi i / R), in place, natural order.
// R = 6 and 12 by the prime-factor maps (Good 1958, Thomas 1963): inputs
// (R2 a + R1 b) mod R, outputs by the Chinese remainders, no twiddles.
// ---------------------------------------------------------------------------
__device__ inline double2 add2(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ inline double2 sub2(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }

__device__ inline void dft3(double2& v0, double2& v1, double2& v2)
{
    constexpr double h = 0.86602540378443864676;  // sin(pi/3)
    const double2 s = add2(v1, v2), d = sub2(v1, v2);
    const double2 t = make_double2(v0.x - 0.5 * s.x, v0.y - 0.5 * s.y);
    v0 = add2(v0, s);
    v1 = make_double2(t.x - h * d.y, t.y + h * d.x);
    v2 = make_double2(t.x + h * d.y, t.y - h * d.x);
}

__device__ inline void dft4(double2& v0, double2& v1, double2& v2, double2& v3)
{
    const double2 a = add2(v0, v2), c = sub2(v0, v2), b = add2(v1, v3), d = sub2(v1, v3);
    v0 = add2(a, b);
    v1 = make_double2(c.x - d.y, c.y + d.x);
    v2 = sub2(a, b);
    v3 = make_double2(c.x + d.y, c.y - d.x);
}

template <int R>
__device__ inline void dft_reg(double2 (&v)[R])
{
    static_assert(R == 3 || R == 4 || R == 5 || R == 6 || R == 8 || R == 12, "no DFT of this length");
    if constexpr (R == 3) {
        dft3(v[0], v[1], v[2]);
    } else if constexpr (R == 4) {
        dft4(v[0], v[1], v[2], v[3]);
    } else if constexpr (R == 5) {
        constexpr double c1 = 0.30901699437494742410, c2 = -0.80901699437494742410;  // cos(2 pi/5), cos(4 pi/5)
        constexpr double s1 = 0.95105651629515357212, s2 = 0.58778525229247312917;   // sin(2 pi/5), sin(4 pi/5)
        const double2 a1 = add2(v[1], v[4]), a2 = add2(v[2], v[3]), d1 = sub2(v[1], v[4]), d2 = sub2(v[2], v[3]);
        const double2 t1 = make_double2(v[0].x + c1 * a1.x + c2 * a2.x, v[0].y + c1 * a1.y + c2 * a2.y);
        const double2 t2 = make_double2(v[0].x + c2 * a1.x + c1 * a2.x, v[0].y + c2 * a1.y + c1 * a2.y);
        const double2 u1 = make_double2(s1 * d1.x + s2 * d2.x, s1 * d1.y + s2 * d2.y);
        const double2 u2 = make_double2(s2 * d1.x - s1 * d2.x, s2 * d1.y - s1 * d2.y);
        v[0] = add2(v[0], add2(a1, a2));
        v[1] = make_double2(t1.x - u1.y, t1.y + u1.x);
        v[4] = make_double2(t1.x + u1.y, t1.y - u1.x);
        v[2] = make_double2(t2.x - u2.y, t2.y + u2.x);
        v[3] = make_double2(t2.x + u2.y, t2.y - u2.x);
    } else if constexpr (R == 8) {
        constexpr double h = 0.70710678118654752440;  // cos(pi/4)
        dft4(v[0], v[2], v[4], v[6]);
        dft4(v[1], v[3], v[5], v[7]);
        const double2 o1 = make_double2(h * (v[3].x - v[3].y), h * (v[3].x + v[3].y));
        const double2 o2 = make_double2(-v[5].y, v[5].x);
        const double2 o3 = make_double2(h * (-v[7].x - v[7].y), h * (v[7].x - v[7].y));
        const double2 e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6], o0 = v[1];
        v[0] = add2(e0, o0);
        v[4] = sub2(e0, o0);
        v[1] = add2(e1, o1);
        v[5] = sub2(e1, o1);
        v[2] = add2(e2, o2);
        v[6] = sub2(e2, o2);
        v[3] = add2(e3, o3);
        v[7] = sub2(e3, o3);
    } else {
        constexpr int R1 = R / 3;  // 2 or 4: inputs (3 a + R1 b) mod R -> outputs a' mod R1, b' mod 3
#pragma unroll
        for (int a = 0; a < R1; ++a) dft3(v[(3 * a) % R], v[(3 * a + R1) % R], v[(3 * a + 2 * R1) % R]);
        double2 w[R];
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            double2 x[R1];
#pragma unroll
            for (int a = 0; a < R1; ++a) x[a] = v[(3 * a + R1 * b) % R];
            if constexpr (R1 == 4) {
                dft4(x[0], x[1], x[2], x[3]);
            } else {
                const double2 s = add2(x[0], x[1]);
                x[1] = sub2(x[0], x[1]);
                x[0] = s;
            }
            // output k with k = a mod R1 and k = b mod 3
#pragma unroll
            for (int k = 0; k < R; ++k)
                if (k % 3 == b) w[k] = x[k % R1];
        }
#pragma unroll
        for (int k = 0; k < R; ++k) v[k] = w[k];
    }
}

// ---------------------------------------------------------------------------
// The plane transforms on square planes of N = RA RB sites a side: the same
// fields, inputs and outputs as k_dft_planes, two radices an axis,
//   y_j[q] = sum_r x[j + RB r] w_RA^(r q),  X[q + RA t] = sum_j w_N^(j q) y_j[q] w_RB^(j t),
// each a DFT in one work-item's registers.  The u axis comes first, so that
// memory is read into registers and written from them in runs of a row; one
// LDS plane (rows of N + 1, so that work-items down a column fall on
// different banks) carries the data between the four steps.  The rows of O
// are real: their plain kernel is the conjugate of the other one's output.
//
// Bound by memory at 48 x 48 (8928 planes: 240 MB read, 330 MB written).  The
// mixed-radix passes of k_dft_planes take three LDS round trips an axis
// through two buffers (two work-groups to a CU, 180 us); here it is three for
// the plane through one buffer (four work-groups to a CU): 124 us, 4.6 TB/s.
// ---------------------------------------------------------------------------
template <int RA, int RB>
constexpr int fft_threads()
{
    return (RA * RB * RB + 63) / 64 * 64;  // one radix-RA butterfly each
}

template <typename ot, int RA, int RB>
__global__ void __launch_bounds__((fft_threads<RA, RB>()), (fft_threads<RA, RB>() >= 512 ? 4 : 3))
    k_fft_planes(const EnsDesc* __restrict__ ens, const int* __restrict__ bstart, int n_ens,
                 const ObsDesc* __restrict__ obs, const int* __restrict__ rlist, const double2* __restrict__ cpl,
                 const ot* __restrict__ opl, const double2* __restrict__ gf, double2* __restrict__ sph,
                 double2* __restrict__ spo)
{
    constexpr int N = RA * RB, S = N + 1, N2 = N * N, T = fft_threads<RA, RB>();
    extern __shared__ __align__(16) unsigned char lds_raw[];
    double2* X = reinterpret_cast<double2*>(lds_raw);  // [N][S]
    double2* tw = X + N * S;
    const int e = find_ens_s(bstart, n_ens, blockIdx.x);
    const EnsDesc& E = ens[e];
    const ObsDesc& O = *obs;
    const int nsig = E.nsig, Si = E.s_in, R = O.n_r, NF = R + 12;
    const int npm = max(E.nx, max(E.ny, E.nz));
    int local = blockIdx.x - bstart[e];
    const int xpar = local % npm;
    local /= npm;
    const int f = local % NF;
    local /= NF;
    const int s = local % Si;
    const int id = local / Si;
    if (id >= O.n_dirs) return;
    const int Np = extent(E, O.dirs[id]);
    if (xpar >= Np) return;  // uniform for the block
    const int tid = threadIdx.x;
    const size_t ps = (size_t)id * Si + s;
    const bool t_field = f < R;
    {
        const int v = tid % N, j = tid / N;
        const bool act = tid < N * RB;
        const int i0 = act ? j * N + v : 0;  // element r: i0 + RB r N
        double2 x[RA];
        if (t_field) {
            const int r = rlist[f];
            const double2* ca = cpl + E.cpl_off + ps * nsig + (size_t)xpar * N2 + i0;
            const double2* cb = cpl + E.cpl_off + ps * nsig + (size_t)((xpar + r) % Np) * N2 + i0;
            const double2* g = gf + E.gf_off + (((size_t)id * R + f) * Si + s) * nsig + (size_t)xpar * N2 + i0;
#pragma unroll
            for (int q = 0; q < RA; ++q) {
                const double2 a = ca[q * RB * N], b = cb[q * RB * N];
                x[q] = cmul(g[q * RB * N], make_double2(a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x));
            }
        } else {
            const ot* op = opl + E.opl_off + (ps * 12 + (f - R)) * nsig + (size_t)xpar * N2 + i0;
#pragma unroll
            for (int q = 0; q < RA; ++q) x[q] = make_double2((double)op[q * RB * N], 0.0);
        }
        for (int i = tid; i < N; i += T) {
            double sn, cs;
            sincospi(2.0 * (double)i / (double)N, &sn, &cs);
            tw[i] = make_double2(cs, sn);
        }
        dft_reg<RA>(x);
        if (act) {
#pragma unroll
            for (int q = 0; q < RA; ++q) X[(q * RB + j) * S + v] = x[q];
        }
    }
    __syncthreads();
    for (int i = tid; i < N * RA; i += T) {  // row q RB + t then holds k1 = q + RA t
        const int v = i % N, q = i / N;
        double2 y[RB];
#pragma unroll
        for (int j = 0; j < RB; ++j) {
            y[j] = X[(q * RB + j) * S + v];
            if (j) y[j] = cmul(y[j], tw[j * q]);
        }
        dft_reg<RB>(y);
#pragma unroll
        for (int t = 0; t < RB; ++t) X[(q * RB + t) * S + v] = y[t];
    }
    __syncthreads();
    {
        const int p = tid % N, j = tid / N;
        const bool act = tid < N * RB;
        double2 x[RA];
        if (act) {
#pragma unroll
            for (int q = 0; q < RA; ++q) x[q] = X[p * S + j + RB * q];
        }
        __syncthreads();  // every column read before the rows are written in another order
        if (act) {
            dft_reg<RA>(x);
#pragma unroll
            for (int q = 0; q < RA; ++q) X[p * S + j * RA + q] = q ? cmul(x[q], tw[j * q]) : x[q];
        }
    }
    __syncthreads();
    double2* out = t_field ? sph + E.sph_off + (ps * R + f) * nsig + (size_t)xpar * N2
                           : spo + E.spo_off + (ps * 12 + (f - R)) * nsig + (size_t)xpar * N2;
    const double sg = t_field ? 1.0 : -1.0;
    for (int i = tid; i < N * RA; i += T) {
        const int q = i % RA, p = i / RA;
        double2 y[RB];
#pragma unroll
        for (int j = 0; j < RB; ++j) y[j] = X[p * S + j * RA + q];
        dft_reg<RB>(y);
        const int k1 = p / RB + RA * (p % RB);
#pragma unroll
        for (int t = 0; t < RB; ++t) out[k1 * N + q + RA * t] = make_double2(y[t].x, sg * y[t].y);
    }
}

// ---------------------------------------------------------------------------
// Spectral sums of one measurement.  Work-group per (ensemble, axis, slab,
// probe group, run of kMacK values of k, kind); the 6 O rows of those k and
// that kind for every x_par are staged in LDS once and shared by all
// separations r:
//   F[...][c][kind][g][k] += sum_{x_par} O^_{row}(x_par + l) (k) * h^~_r(x_par) (k)
// with l = l_g + (mode_g ? l_mid(r, c) : 0) and row = 2 o(c, axis) + kind.
// Work-item (k, r slot) takes r = slot, slot + kMacThreads / kMacK, ...  Every
// sum runs over x_par in ascending order.
//
// Bound by the latency of its loads: 48^3 x 12 with 19 separations moves 430
// MB.
// So the O rows go straight from memory to LDS (global_load_lds), all in
// flight together with the first T spectra and the running sums; the T
// spectra then come in two register buffers of kMacAhead values, one summed
// while the other loads (8 or 12 instead of 6: the same within noise); and a
// work-group holds one kind, so that four fit a CU's LDS instead of two (the
// kinds of a tile share the T spectra through the L2 of their XCD: memory
// reads stay the same).  NC, the number of components, is a constant, so that
// no branch separates the LDS reads of one position from the next.  240 us
// with the O rows of both kinds staged through registers and every load
// awaited where it was used, 152 us with copies and buffers, 140 us now
// (3.1 TB/s).
// ---------------------------------------------------------------------------
constexpr int kMacAhead = 6;

template <int NC>
__global__ void __launch_bounds__(kMacThreads, 3) k_spec_mac(const EnsDesc* __restrict__ ens,
                                                             const int* __restrict__ bstart, int n_ens,
                                                             const ObsDesc* __restrict__ obs,
                                                             const int* __restrict__ rlist, const int* __restrict__ comps,
                                                             const int* __restrict__ gdesc, const double2* __restrict__ sph,
                                                             const double2* __restrict__ spo, double2* __restrict__ facc,
                                                             int tile0, int n_tiles)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    double2* os = reinterpret_cast<double2*>(lds_raw);  // [orientation][x_par][kk]
    constexpr int KC = kMacK, A = kMacAhead;
    // the two kinds of a tile eight work-groups apart: the same XCD, whose L2 then holds the T spectra for both
    const int kind = (blockIdx.x >> 3) & 1, tile = tile0 + (int)(blockIdx.x & 7u) + (int)(blockIdx.x >> 4) * 8;
    if (tile >= n_tiles) return;  // uniform: padding of the launch to a multiple of 16
    const int e = find_ens_s(bstart, n_ens, tile);
    const EnsDesc& E = ens[e];
    const ObsDesc& O = *obs;
    const int nsig = E.nsig, Si = E.s_in, R = O.n_r, NG = O.n_groups;
    int n12max = 0;
    for (int i = 0; i < O.n_dirs; ++i) n12max = max(n12max, nsig / extent(E, O.dirs[i]));
    const int nkc = (n12max + KC - 1) / KC;
    int local = tile - bstart[e];
    const int kc = local % nkc;
    local /= nkc;
    const int g = local % NG;
    local /= NG;
    const int s = local % Si;
    const int id = local / Si;
    if (id >= O.n_dirs) return;
    const int dir = O.dirs[id];
    const int N = extent(E, dir), n12 = nsig / N;
    const int k0 = kc * KC;
    if (k0 >= n12) return;  // uniform for the block
    const size_t ps = (size_t)id * Si + s;
    const int kk = threadIdx.x % KC, slot = threadIdx.x / KC;
    const int k = min(k0 + kk, n12 - 1);  // past the plane's end: a copy of the last k, not stored
    // element i = (orientation N + x_par) KC + kk of the tile: 64 consecutive ones per wave and round
    {
        const double2* src = spo + E.spo_off + (ps * 12 + kind) * nsig + k;
        const int n_os = 6 * N * KC, lane = threadIdx.x & 63;
        for (int j = (int)threadIdx.x & ~63; j < n_os; j += kMacThreads) {
            const int i = j + lane;
            if (i < n_os) {  // lane % KC is kk: KC divides 64
                const int t = i / KC, o = t / N;
                __builtin_amdgcn_global_load_lds((const void*)(src + (size_t)(t + o * N) * n12),
                                                 (__attribute__((address_space(3))) void*)(os + j), 16, 0, 0);
            }
        }
    }
    const int wrap = N * KC;
    bool first = true;
    for (int ir = slot; ir < R || first; ir += kMacThreads / KC) {
        const bool act = ir < R;  // the first round has every work-item, for the barrier
        const int irc = act ? ir : R - 1;
        const int r = rlist[irc];
        const double2* h = sph + E.sph_off + (ps * R + irc) * nsig + k;
        double2 b0[A], b1[A];
        auto fetch = [&](double2(&b)[A], int x0) {
#pragma unroll
            for (int u = 0; u < A; ++u) b[u] = h[(size_t)min(x0 + u, N - 1) * n12];
        };
        fetch(b0, 0);
        const size_t sl0 = ((ps * R + irc) * NC * 2 + kind) * NG + g;
        double2* F = facc + E.facc_off + sl0 * n12max + k;
        const size_t fstep = 2 * (size_t)NG * n12max;
        double2 f[NC];
#pragma unroll
        for (int ic = 0; ic < NC; ++ic) f[ic] = F[(size_t)ic * fstep];
        // LDS offsets of O at x_par + l: xa for components that lie across the axis, xb for those that span it
        const int lg = gdesc[2 * g], mid = gdesc[2 * g + 1];
        int xa = ((((lg + (mid ? r / 2 : 0)) % N) + N) % N) * KC + kk;
        int xb = ((((lg + (mid ? (r - 1) / 2 : 0)) % N) + N) % N) * KC + kk;
        int ob[NC], span[NC];  // span: all bits set or none
        double re[NC], im[NC];
#pragma unroll
        for (int ic = 0; ic < NC; ++ic) {
            const int c = comps[ic];
            span[ic] = spans_axis(c) ? -1 : 0;
            ob[ic] = orient_of(c, dir) * wrap;
            re[ic] = im[ic] = 0.0;
        }
        auto sum = [&](const double2& b) {
            const int dx = xb - xa;
#pragma unroll
            for (int ic = 0; ic < NC; ++ic) {
                const double2 a = os[ob[ic] + xa + (dx & span[ic])];
                re[ic] += a.x * b.x - a.y * b.y;
                im[ic] += a.x * b.y + a.y * b.x;
            }
            xa += KC;
            xb += KC;
            if (xa >= wrap) xa -= wrap;
            if (xb >= wrap) xb -= wrap;
        };
        if (first) {
            __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wave's copies into LDS have landed
            __syncthreads();
            first = false;
        }
        int x0 = 0;
        for (; x0 + 2 * A <= N; x0 += 2 * A) {
            fetch(b1, x0 + A);
#pragma unroll
            for (int u = 0; u < A; ++u) sum(b0[u]);
            fetch(b0, x0 + 2 * A);
#pragma unroll
            for (int u = 0; u < A; ++u) sum(b1[u]);
        }
        fetch(b1, x0 + A);
#pragma unroll
        for (int u = 0; u < A; ++u)
            if (x0 + u < N) sum(b0[u]);
#pragma unroll
        for (int u = 0; u < A; ++u)
            if (x0 + A + u < N) sum(b1[u]);
        if (!act || k0 + kk >= n12) continue;
#pragma unroll
        for (int ic = 0; ic < NC; ++ic) F[(size_t)ic * fstep] = make_double2(f[ic].x + re[ic], f[ic].y + im[ic]);
    }
}

// ---------------------------------------------------------------------------
// Probe estimates of the configuration.  Work-group per (ensemble, r,
// component, kind, probe group); its probes p have
//   CO = scale sum_axis 1/(n1 n2) sum_k1 e^(2 pi i k1 p1/n1) A(k1, p2),
//   A(k1, v) = sum_k2 F(k1, k2) e^(2 pi i k2 v/n2),  F(k) = sum_s F[axis][s][r][c][kind][g][k],
// scale = 1/(N_sigma |M| N_t n_o n_i).  Each of the three sums runs in double-
// double in ascending order, its products with the twiddles exact, and F and A
// are held as pairs (hi, lo): the rounding of the twiddles is all that differs
// from the exact sum of the spectra.  A's rows replace F's in LDS as they are
// formed, so the pairs take the space of one plane of each.
//
// A probe by itself needs n1 n2 terms of every slab; the slabs first, then the
// rows at the nv positions p2 that the group's probes have, then the columns
// take n1 n2 (S + nv) per work-group and n1 per probe.  48^3 x 12 with 441
// probes and 19 separations: 13 million terms instead of 600 million, 3.44 ms
// before and 65 us now (57 us with F and A rounded to one double each, 1.2 to
// 1.4 times the error).  The rows' chains of double-double sums bound it, so
// two work-groups per CU: two values of A per work-item and one loop for both
// tables of twiddles keep it at 128 registers without spills (four values and
// rows at every position: 166, one work-group, 97 us).  A configuration of
// 48^3 x 4 with 63 probes takes 622 us (931 us).
// ---------------------------------------------------------------------------
constexpr int kFinalThreads = 512;
constexpr int kFinalRow = 2;  // values of A per work-item and pass over the rows
constexpr int kFinalExtent = 128;  // largest extent (k_spec_mac's LDS holds up to 106)

// hi + lo += b, hi the rounded running sum, lo the sum of its errors
__device__ inline void pair_add(double& hi, double& lo, double b)
{
    const double s = hi + b, t = s - hi;
    lo += (hi - (s - t)) + (b - t);
    hi = s;
}

struct cpair {
    double2 hi, lo;
    // += f w, f = fh + fl; the products of fh exact
    __device__ inline void add_mul(double2 fh, double2 fl, double2 w)
    {
        const double p0 = fh.x * w.x, p1 = fh.y * w.y, p2 = fh.x * w.y, p3 = fh.y * w.x;
        pair_add(hi.x, lo.x, p0);
        pair_add(hi.x, lo.x, -p1);
        pair_add(hi.y, lo.y, p2);
        pair_add(hi.y, lo.y, p3);
        lo.x += (fma(fh.x, w.x, -p0) - fma(fh.y, w.y, -p1)) + (fl.x * w.x - fl.y * w.y);
        lo.y += (fma(fh.x, w.y, -p2) + fma(fh.y, w.x, -p3)) + (fl.x * w.y + fl.y * w.x);
    }
    __device__ inline void norm()
    {
        const double x = hi.x + lo.x, y = hi.y + lo.y;
        lo = make_double2(lo.x - (x - hi.x), lo.y - (y - hi.y));
        hi = make_double2(x, y);
    }
};

// A's rows from k1 = row0 on at the nv positions v[], n values in all (n <= U
// kFinalThreads), over F's
template <int U>
__device__ inline void final_rows(double2* Fh, double2* Fl, const double2* w, const int* vs, int nv, int n2, int row0, int n)
{
    cpair a[U];
    int f[U], j[U], v[U], ph[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int i = min((int)threadIdx.x + u * kFinalThreads, n - 1), row = i / nv;
        f[u] = (row0 + row) * n2;
        j[u] = i - row * nv;
        v[u] = vs[j[u]];
        ph[u] = 0;
        a[u] = cpair{make_double2(0.0, 0.0), make_double2(0.0, 0.0)};
    }
    for (int k2 = 0; k2 < n2; ++k2)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            a[u].add_mul(Fh[f[u] + k2], Fl[f[u] + k2], w[ph[u]]);
            ph[u] += v[u];
            if (ph[u] >= n2) ph[u] -= n2;
        }
    __syncthreads();  // these rows of F have been read
#pragma unroll
    for (int u = 0; u < U; ++u)
        if ((int)threadIdx.x + u * kFinalThreads < n) {
            a[u].norm();
            Fh[f[u] + j[u]] = a[u].hi;
            Fl[f[u] + j[u]] = a[u].lo;
        }
}

__global__ void __launch_bounds__(kFinalThreads, 4) k_spec_final(const EnsDesc* __restrict__ ens, unsigned sum0,
                                                              const ObsDesc* __restrict__ obs,
                                                              const int* __restrict__ probes,
                                                              const int* __restrict__ pgroup,
                                                              const double2* __restrict__ facc, double n_meas_total,
                                                              double* __restrict__ results, const int* __restrict__ ring)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    __shared__ int wanted[kFinalExtent], vs[kFinalExtent];  // whether a position v is a probe's, and those positions
    const ObsDesc& O = *obs;
    const int R = O.n_r, Np = O.n_probe, Nc = O.n_comp, NG = O.n_groups;
    const unsigned sum = sum0 + blockIdx.x;  // (((e R + ir) Nc + ic) 2 + kind) NG + g
    const int g = (int)(sum % (unsigned)NG);
    const unsigned t = sum / (unsigned)NG;
    const int rck = (int)(t % (unsigned)(R * Nc * 2)), e = (int)(t / (unsigned)(R * Nc * 2));
    const int ir = rck / (Nc * 2), ck = rck - ir * Nc * 2;
    const EnsDesc& E = ens[e];
    const int nsig = E.nsig, Si = E.s_in;
    int n12max = 0;
    for (int i = 0; i < O.n_dirs; ++i) n12max = max(n12max, nsig / extent(E, O.dirs[i]));
    const int npm = max(E.nx, max(E.ny, E.nz));
    double2* Fh = reinterpret_cast<double2*>(lds_raw);
    double2* Fl = Fh + n12max;
    double2* w1 = Fl + n12max;
    double2* w2 = w1 + npm;
    const double scale = 1.0 / ((double)nsig * O.n_dirs * E.nt * n_meas_total);
    double* out = results + ((size_t)(*ring) * O.n_ens_total + E.res_index) * O.n_doubles_per_config + 2ll * R;
    for (int p0 = 0; p0 < Np; p0 += kFinalThreads) {  // as many probes as work-items, usually all
        const int p = p0 + (int)threadIdx.x;
        const bool mine = p < Np && pgroup[min(p, Np - 1)] == g;
        const int p1 = mine ? probes[4 * p + 1] : 0, p2 = mine ? probes[4 * p + 2] : 0;
        dds are{0.0, 0.0}, aim{0.0, 0.0};
        for (int id = 0; id < O.n_dirs; ++id) {
            const int dir = O.dirs[id];
            const int n1 = extent(E, dir == 2 ? 0 : dir + 1), n2 = extent(E, dir == 0 ? 2 : dir - 1), n12 = n1 * n2;
            const int q1 = ((p1 % n1) + n1) % n1, q2 = ((p2 % n2) + n2) % n2;
            __syncthreads();  // the previous axis is done with the tables
            if (threadIdx.x < kFinalExtent) wanted[threadIdx.x] = 0;
            __syncthreads();
            if (mine) wanted[q2] = 1;
            for (int i = threadIdx.x; i < n1 + n2; i += kFinalThreads) {
                const bool first = i < n1;
                const int j = first ? i : i - n1;
                double sn, cs;
                sincospi(2.0 * (double)j / (double)(first ? n1 : n2), &sn, &cs);
                (first ? w1 : w2)[j] = make_double2(cs, sn);
            }
            const size_t sstep = (size_t)R * Nc * 2 * NG * n12max;  // from one slab to the next
            const double2* Fg = facc + E.facc_off + ((((size_t)id * Si * R + ir) * Nc * 2 + ck) * NG + g) * n12max;
            for (int k = threadIdx.x; k < n12; k += kFinalThreads) {
                dds re{0.0, 0.0}, im{0.0, 0.0};
#pragma unroll 4
                for (int s = 0; s < Si; ++s) {
                    const double2 v = Fg[s * sstep + k];
                    re = dds_add(re, v.x);
                    im = dds_add(im, v.y);
                }
                Fh[k] = make_double2(re.hi, im.hi);
                Fl[k] = make_double2(re.lo, im.lo);
            }
            __syncthreads();
            // the wanted positions, two ballots of a wave (extents are at most 106)
            const int lane = (int)threadIdx.x & 63;
            const unsigned long long lo = __ballot(wanted[lane] != 0), hi = __ballot(wanted[64 + lane] != 0);
            const int nlo = __popcll(lo), nv = nlo + __popcll(hi);
            auto place = [&](int v) {
                return v < 64 ? __popcll(lo & ((1ull << v) - 1)) : nlo + __popcll(hi & ((1ull << (v - 64)) - 1));
            };
            if (threadIdx.x < kFinalExtent && wanted[threadIdx.x]) vs[place((int)threadIdx.x)] = (int)threadIdx.x;
            __syncthreads();
            // whole rows a pass
            const int rows = nv ? kFinalRow * kFinalThreads / nv : n1;
            for (int k1 = 0; nv && k1 < n1; k1 += rows) {
                const int n = min(rows, n1 - k1) * nv;
                if (n <= kFinalThreads)
                    final_rows<1>(Fh, Fl, w2, vs, nv, n2, k1, n);
                else
                    final_rows<kFinalRow>(Fh, Fl, w2, vs, nv, n2, k1, n);
            }
            __syncthreads();
            if (!mine) continue;
            const int at = place(q2);
            cpair a{make_double2(0.0, 0.0), make_double2(0.0, 0.0)};
            int ph = 0;
            for (int k1 = 0; k1 < n1; ++k1) {
                a.add_mul(Fh[k1 * n2 + at], Fl[k1 * n2 + at], w1[ph]);
                ph += q1;
                if (ph >= n1) ph -= n1;
            }
            a.norm();
            const double n = (double)n12;  // a / n as a pair: the quotient and its remainder's
            const double qx = a.hi.x / n, qy = a.hi.y / n;
            are = dds_add(dds_add(are, qx), (fma(-qx, n, a.hi.x) + a.lo.x) / n);
            aim = dds_add(dds_add(aim, qy), (fma(-qy, n, a.hi.y) + a.lo.y) / n);
        }
        if (!mine) continue;
        const size_t idx = ((size_t)ir * Np + p) * Nc * 2 + ck;
        out[2 * idx] = (are.hi + are.lo) * scale;
        out[2 * idx + 1] = (aim.hi + aim.lo) * scale;
    }
}

// element copy in 16-byte units (the replay's copy of the links; a kernel so
// that captured graphs hold no memset or memcpy nodes)
__global__ void k_copy16(const uint4* __restrict__ src, uint4* __restrict__ dst, size_t n16)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (size_t)gridDim.x * blockDim.x)
        dst[i] = src[i];
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
hipError_t launch_wfac(const EnsDesc* d_ens, const int* d_bstart, int n_ens, int total_blocks, const ObsDesc* d_obs,
                       const double2* out_t, double scale, double2* wf, const double* results, const int* d_ring,
                       hipStream_t st)
{
    hipLaunchKernelGGL(k_wfac, dim3(total_blocks), dim3(256), 0, st, d_ens, d_bstart, n_ens, d_obs, out_t, scale, wf,
                       results, d_ring);
    return hipGetLastError();
}

hipError_t launch_gfac(const EnsDesc* d_ens, const int* d_bstart, int n_ens, int total_blocks, const ObsDesc* d_obs,
                       const double2* avg_t, const double2* wf, int q, double2* gf, const double* results,
                       const int* d_ring, hipStream_t st)
{
    hipLaunchKernelGGL(k_gfac, dim3(total_blocks), dim3(256), 0, st, d_ens, d_bstart, n_ens, d_obs, avg_t, wf, q, gf,
                       results, d_ring);
    return hipGetLastError();
}

// tile: 4 when every transverse extent is a multiple of 4, else 2 (extents are even)
hipError_t launch_plane_stage(const EnsDesc* d_ens, const int* d_bstart, int n_ens, int total_blocks,
                              const ObsDesc* d_obs, const double2* hist_c, const void* hist_o, int m_in,
                              int precision, double2* cpl, void* opl, hipStream_t st)
{
    if (total_blocks <= 0) return hipSuccess;
    if (precision == 0)
        hipLaunchKernelGGL(k_plane_stage<double>, dim3(total_blocks), dim3(kStageTile * kStageTile), 0, st, d_ens, d_bstart, n_ens, d_obs,
                           hist_c, (const double*)hist_o, m_in, cpl, (double*)opl);
    else
        hipLaunchKernelGGL(k_plane_stage<float>, dim3(total_blocks), dim3(kStageTile * kStageTile), 0, st, d_ens, d_bstart, n_ens, d_obs,
                           hist_c, (const float*)hist_o, m_in, cpl, (float*)opl);
    return hipGetLastError();
}

// sides with a transform in registers and their radices
#define U1ML_FFT_SIDES(X)                                                                                              \
    X(4, 3) X(4, 4) X(6, 3) X(5, 4) X(6, 4) X(6, 5) X(8, 4) X(6, 6) X(8, 5) X(12, 4) X(12, 5) X(8, 8)

bool fft_in_registers(int side)
{
#define U1ML_FFT(RA, RB)                                                                                               \
    if (side == RA * RB) return true;
    U1ML_FFT_SIDES(U1ML_FFT)
#undef U1ML_FFT
    return false;
}

// square: the side of every plane of the launch, 0 if they differ or are not square; n12max, npm: largest plane and extent
hipError_t launch_dft_planes(const EnsDesc* d_ens, const int* d_bstart, int n_ens, int total_blocks, int square,
                             int n12max, int npm, const ObsDesc* d_obs, const int* d_r, const double2* cpl,
                             const void* opl, const double2* gf, double2* sph, double2* spo, int precision, int tile,
                             hipStream_t st)
{
    // Square planes of one size whose side has two radices take the transform
    // in registers (48 x 48: 124 instead of 180 us); every other plane the
    // mixed-radix passes or, with a prime factor above 5, the direct sums.
    if (square > 0) {
        const size_t lds = (size_t)square * (square + 2) * 16;
#define U1ML_FFT(RA, RB)                                                                                               \
    case RA * RB:                                                                                                      \
        if (precision == 0)                                                                                            \
            hipLaunchKernelGGL((k_fft_planes<double, RA, RB>), dim3(total_blocks), dim3(fft_threads<RA, RB>()), lds,   \
                               st, d_ens, d_bstart, n_ens, d_obs, d_r, cpl, (const double*)opl, gf, sph, spo);         \
        else                                                                                                           \
            hipLaunchKernelGGL((k_fft_planes<float, RA, RB>), dim3(total_blocks), dim3(fft_threads<RA, RB>()), lds,    \
                               st, d_ens, d_bstart, n_ens, d_obs, d_r, cpl, (const float*)opl, gf, sph, spo);          \
        return hipGetLastError();
        switch (square) {
            U1ML_FFT_SIDES(U1ML_FFT)
        }
#undef U1ML_FFT
    }
    const dim3 g(total_blocks), b(kPlaneThreads);
    const size_t lds_bytes = plane_lds(n12max, npm);
    if (precision == 0) {
        if (tile == 4)
            hipLaunchKernelGGL((k_dft_planes<double, 4>), g, b, lds_bytes, st, d_ens, d_bstart, n_ens, d_obs, d_r,
                               cpl, (const double*)opl, gf, sph, spo);
        else
            hipLaunchKernelGGL((k_dft_planes<double, 2>), g, b, lds_bytes, st, d_ens, d_bstart, n_ens, d_obs, d_r,
                               cpl, (const double*)opl, gf, sph, spo);
    } else {
        if (tile == 4)
            hipLaunchKernelGGL((k_dft_planes<float, 4>), g, b, lds_bytes, st, d_ens, d_bstart, n_ens, d_obs, d_r,
                               cpl, (const float*)opl, gf, sph, spo);
        else
            hipLaunchKernelGGL((k_dft_planes<float, 2>), g, b, lds_bytes, st, d_ens, d_bstart, n_ens, d_obs, d_r,
                               cpl, (const float*)opl, gf, sph, spo);
    }
    return hipGetLastError();
}

hipError_t launch_spec_mac(const EnsDesc* d_ens, const int* d_bstart, int n_ens, int total_blocks, int npm,
                           int n_comp, const ObsDesc* d_obs, const int* d_r, const int* d_comp, const int* d_gdesc,
                           const double2* sph, const double2* spo, double2* facc, hipStream_t st)
{
    if (total_blocks <= 0) return hipSuccess;
    const size_t lds = spec_mac_lds(npm);
    for (int t0 = 0; t0 < total_blocks; t0 += (int)kMaxGrid) {  // usually one
        const dim3 gr((std::min(total_blocks - t0, (int)kMaxGrid) + 7) / 8 * 16), bl(kMacThreads);
#define U1ML_MAC(NC)                                                                                                   \
    case NC:                                                                                                           \
        hipLaunchKernelGGL(k_spec_mac<NC>, gr, bl, lds, st, d_ens, d_bstart, n_ens, d_obs, d_r, d_comp, d_gdesc, sph,  \
                           spo, facc, t0, total_blocks);                                                               \
            break;
        switch (n_comp) {
            case 0: return hipSuccess;
            U1ML_MAC(1)
            U1ML_MAC(2)
            U1ML_MAC(3)
            U1ML_MAC(4)
            U1ML_MAC(5)
            U1ML_MAC(6)
            default: return hipErrorInvalidValue;
        }
#undef U1ML_MAC
    }
    return hipGetLastError();
}

// n_sums: sums per ensemble (n_r n_comp 2 n_groups); npm, n12max: largest lattice extent and plane
hipError_t launch_spec_final(const EnsDesc* d_ens, int n_ens, const ObsDesc* d_obs, long long n_sums, int npm,
                             int n12max, const int* d_probe, const int* d_pgroup, const double2* facc,
                             double n_meas_total, double* results, const int* d_ring, hipStream_t st)
{
    if (n_sums <= 0) return hipSuccess;
    const long long all = n_sums * n_ens;
    for (long long s0 = 0; s0 < all; s0 += kMaxGrid)  // usually one
        hipLaunchKernelGGL(k_spec_final, dim3((unsigned)std::min<long long>(all - s0, kMaxGrid)), dim3(kFinalThreads),
                           plane_lds(n12max, npm), st, d_ens, (unsigned)s0, d_obs, d_probe, d_pgroup, facc,
                           n_meas_total, results, d_ring);
    return hipGetLastError();
}

hipError_t launch_copy(const void* src, void* dst, size_t bytes, hipStream_t st)
{
    const size_t n16 = bytes / 16;
    if (n16 == 0) return hipSuccess;
    size_t g = (n16 + 255) / 256;
    if (g > 8192) g = 8192;
    hipLaunchKernelGGL(k_copy16, dim3((unsigned)g), dim3(256), 0, st, (const uint4*)src, (uint4*)dst, n16);
    return hipGetLastError();
}

}  // namespace u1ml
