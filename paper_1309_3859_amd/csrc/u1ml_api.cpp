// u1ml_api.cpp -- host side of libu1ml: planner, workspace layout, the
// Algorithm-1 scheduler (Amado, Cardoso, Bicudo, arXiv 1309.3859, Sec. II.C)
// with HIP-graph capture, and the C ABI declared in include/u1ml.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <map>
#include <memory>
#include <string>
#include <utility>
#include <vector>

#include "../../include/u1ml.h"
#include "u1ml_internal.hpp"

using namespace u1ml;

namespace {

thread_local std::string g_err;  // context-free error text

constexpr size_t kAlign = 256;

inline size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

bool mul_ok(size_t a, size_t b, size_t* out) { return !__builtin_mul_overflow(a, b, out); }
bool add_ok(size_t a, size_t b, size_t* out) { return !__builtin_add_overflow(a, b, out); }

struct Sizes {
    // per ensemble element offsets
    std::vector<size_t> links, hc, ho, at, ato, ot, oto, vac, hit;
    std::vector<size_t> wf, gf, sph, spo, facc;  // spectral form (double2 elements)
    std::vector<size_t> cpl, opl;                // plane-major copies (double2, real elements)
};

struct Layout {
    size_t off_links, off_hc, off_ho, off_at, off_ato, off_ot, off_oto, off_res, off_scr;
    size_t sz_links, sz_hc, sz_ho, sz_at, sz_ato, sz_ot, sz_oto, sz_res, sz_scr;
    // spectral form: weights W, G; plane spectra of T and O; spectral sums; replay copy of the links
    size_t off_wf, off_gf, off_sph, off_spo, off_facc, off_saved, off_cpl, off_opl;
    size_t sz_wf, sz_gf, sz_sph, sz_spo, sz_facc, sz_saved, sz_cpl, sz_opl;
    // scratch sub-offsets (bytes from off_scr)
    size_t s_ens, s_obs, s_r, s_probe, s_comp, s_bstart, s_upd, s_ring, s_vpart, s_ppart, s_pout, s_count,
        s_stage, s_bmap, s_mmap, s_prodpart, s_pgroup, s_gdesc, s_pblk, s_prow, s_pmap[kPairClasses], s_smap[3], s_hit;
    size_t off_alt;  // the other link buffer (both-parities updates)
    // the lanes' descriptors and tables (each sized for the whole batch)
    size_t s_lens[4], s_lbstart[4], s_lbmap[4], s_lmmap[4], s_lring[4], s_lpmap[4][kPairClasses], s_lsmap[4][3];
    size_t bmap_stride;  // entries per update class (blocks of 64 threads)
    int n_bstart_tables;
};

constexpr int kTabUpd = 0;    // 4 update classes
constexpr int kTabAll = 4;    // all links (init, health)
constexpr int kTabMeas = 5;   // spatial sites
constexpr int kTabCon = 6;    // contraction items
constexpr int kTabComb = 7;   // combine items
constexpr int kTabProd = 8;   // slab-product work-groups
constexpr int kTabSite = 9;   // spectral weights: (axis, r, site) items
constexpr int kTabPlane = 10; // spectral plane transforms: work-groups
constexpr int kTabMac = 11;   // spectral sums: work-groups
constexpr int kTabStage = 12; // spectral staging: work-groups
constexpr int kTabIns = 13;   // insertion contraction: work-groups
constexpr int kNumTabs = 14;
constexpr int kXcds = 8;  // accelerator complex dies of an MI355X, each with its own L2
constexpr int kMaxLanes = 4;  // streams that sweeps and configurations are spread over
// Lanes a context starts with, by the batch's sites: two where a phase of half
// the batch still fills the device, else one (a second stream costs more than
// its overlap gains, and more than two never gain).  MI355X, us per sweep, full /
// inside slabs, 1 lane and 2 lanes: FP32 8 x 24^3 x 8 (0.88M sites) 147 / 111, 158 /
// 133; 32 x 16^3 x 8 (1.05M) 161 / 120, 151 / 119; 256 x 8^3 x 8 160 / 72, 154 / 74;
// 16 x 24^3 x 8 (1.77M) 225 / 165, 193 / 157; FP64 8 x 24^3 x 4 (0.44M) 214 / 158, 193 /
// 169; 16 x 16^3 x 8 (0.52M) 218 / 160, 195 / 154; 8 x 24^3 x 8 303 / 235, 288 / 220.
int default_lanes(const std::vector<u1ml_ensemble>& ens, int precision)
{
    double sites = 0.0;
    for (const u1ml_ensemble& E : ens) sites += (double)E.ns[0] * E.ns[1] * E.ns[2] * E.nt;
    return ens.size() > 1 && sites >= (precision == U1ML_FP64 ? 0.5e6 : 1.0e6) ? 2 : 1;
}

// Tile of a both-parities launch (k_pair): core rows along y, z, t.
struct PairTile {
    int L[3] = {0, 0, 0};
    long long blocks = 0;
};

struct Problem {
    int n_ens = 0;
    std::vector<u1ml_ensemble> ens;
    int precision = 0, n_or = 3, n_levels = 1;
    u1ml_level lv[2] = {};
    int n_dirs = 1;
    int dirs[3] = {0, 0, 0};
    std::vector<int> r;
    std::vector<u1ml_probe> probes;
    std::vector<int> comps;
    int max_configs = 1;
    int form_req = U1ML_FORM_AUTO;
    int update = U1ML_UPDATE_HEATBATH;
    bool multihit = false;
    int ins_kernel = 0;  // 0: estimated faster, 1: vector, 2: matrix cores
    double metro_delta = 1.0;
    // derived
    int tau_i = 2, n_i = 1, k_i = 1, tau_o = 2, n_o = 1, k_o = 0;
    bool two = false;
    bool spectral = false;        // insertion contraction in the spectral form
    double est_hist_ms = 0.0, est_spec_ms = -1.0;  // the planner's cost estimates of the two forms
    std::vector<int> pgroup;      // probe -> group of probes sharing (l, mode)
    std::vector<int> gdesc;       // group -> (l, mode)
    std::vector<int> pblk;        // insertion contraction: slot blocks, kInsBlkInts ints each
    int ins_ks = 1;               // insertion contraction: slots per block (kMfSlots: matrix cores)
    // insertion slot keys: (l, mode, spans) and their (probe, component index) slots
    std::vector<std::vector<std::pair<int, int>>> skeys;
    std::vector<int> skey_l, skey_mode, skey_spans;
    int ins_ks_vec = 1;           // the vector kernel's slots per block
    bool ins_mfma_est = false;    // the matrix-core kernel is estimated faster (and applies)
    long long nd_cfg = 0;
    // both-parities launches: per class whether sweeps use them, the ensembles' tiles, the work-group
    // size; the row tables of every tile shape
    bool pair_on[kPairClasses] = {};
    int pair_block[kPairClasses] = {};
    std::vector<PairTile> pair_tile[kPairClasses];
    int n_pair_rows = 0;
    std::map<std::array<int, 15>, int> pair_shape;  // shape -> first row
    std::vector<int> lattice;  // per ensemble: the first one of its extents

    // whole sweeps in LDS (k_slab), per class full / inner tau / outer tau: on, work-group size, LDS, work-groups
    bool slab_on[3] = {};
    int slab_block[3] = {};
    size_t slab_lds_bytes[3] = {};
    size_t slab_blocks[3] = {};

    bool any_pair() const { return std::find(pair_on, pair_on + kPairClasses, true) != pair_on + kPairClasses; }
    // time slices per slab whose links a class updates at thickness tau, and slabs (temporal or full: all, one)
    int pair_tau(int cls) const { return cls == 9 || cls % 3 == 0 ? 0 : (cls % 3 == 1 ? tau_i : tau_o); }
};

// frame components whose plaquette spans the charge axis: E_par (P_{par t}),
// B_perp1 (P_{perp2 par}) and B_perp2 (P_{par perp1})
bool comp_spans_axis_host(int c) { return c == 0 || c == 4 || c == 5; }

bool fail(std::string* err, const std::string& msg)
{
    if (err) *err = msg;
    return false;
}

// slot blocks of ks slots (kInsBlkInts ints each): l, mode, spans, number of
// slots, then per slot probe, component index, p1, p2
void pack_slot_blocks(Problem* P, int ks)
{
    P->pblk.clear();
    P->ins_ks = ks;
    for (size_t kk = 0; kk < P->skeys.size(); ++kk) {
        const auto& key = P->skeys[kk];
        for (size_t b = 0; b < key.size(); b += ks) {
            int blk[kInsBlkInts] = {};
            blk[0] = P->skey_l[kk];
            blk[1] = P->skey_mode[kk];
            blk[2] = P->skey_spans[kk];
            blk[3] = (int)std::min<size_t>(ks, key.size() - b);
            for (int k = 0; k < blk[3]; ++k) {
                const int p = key[b + k].first, ic = key[b + k].second;
                blk[4 + 4 * k] = p;
                blk[5 + 4 * k] = ic;
                blk[6 + 4 * k] = P->probes[p].p1;
                blk[7 + 4 * k] = P->probes[p].p2;
            }
            P->pblk.insert(P->pblk.end(), blk, blk + kInsBlkInts);
        }
    }
}

bool read_problem(const u1ml_problem* p, Problem* P, std::string* err)
{
    if (!p) return fail(err, "problem is NULL");
    if (p->n_ens < 1 || !p->ens) return fail(err, "n_ens must be >= 1 with a non-NULL ensemble array");
    if (p->precision != U1ML_FP64 && p->precision != U1ML_FP32) return fail(err, "precision must be 0 (FP64) or 1 (FP32)");
    if (p->n_or < 0) return fail(err, "n_or must be >= 0");
    if (p->update != U1ML_UPDATE_HEATBATH && p->update != U1ML_UPDATE_METROPOLIS)
        return fail(err, "update must be 0 (heatbath) or 1 (Metropolis)");
    if (p->update == U1ML_UPDATE_METROPOLIS && !(p->metro_delta > 0.0 && p->metro_delta <= M_PI))
        return fail(err, "metro_delta must satisfy 0 < delta <= pi");
    P->update = p->update;
    if (p->multihit != 0 && p->multihit != 1) return fail(err, "multihit must be 0 or 1");
    P->multihit = p->multihit == 1;
    if (p->ins_kernel < 0 || p->ins_kernel > 2) return fail(err, "ins_kernel must be 0, 1 or 2");
    P->ins_kernel = p->ins_kernel;
    P->metro_delta = p->metro_delta;
    if (p->n_levels < 1 || p->n_levels > 2) return fail(err, "n_levels must be 1 or 2");
    if (p->max_configs < 1) return fail(err, "max_configs must be >= 1");
    P->n_ens = p->n_ens;
    P->ens.assign(p->ens, p->ens + p->n_ens);
    P->precision = p->precision;
    P->n_or = p->n_or;
    P->n_levels = p->n_levels;
    P->lv[0] = p->levels[0];
    P->lv[1] = p->levels[1];
    P->max_configs = p->max_configs;
    for (int k = 0; k < p->n_levels; ++k) {
        const u1ml_level& L = p->levels[k];
        if (L.tau < 2) return fail(err, "level tau must be >= 2 (a slab needs a frozen boundary layer)");
        if (L.n_iter < 1) return fail(err, "level n_iter must be >= 1");
        if (L.k_sweeps < 0) return fail(err, "level k_sweeps must be >= 0");
    }
    P->two = (p->n_levels == 2);
    if (P->two) {
        P->tau_o = p->levels[0].tau;
        P->n_o = p->levels[0].n_iter;
        P->k_o = p->levels[0].k_sweeps;
        P->tau_i = p->levels[1].tau;
        P->n_i = p->levels[1].n_iter;
        P->k_i = p->levels[1].k_sweeps;
        if (P->tau_o % P->tau_i != 0) return fail(err, "outer tau must be a multiple of the inner tau");
        if (P->tau_o / P->tau_i > 8) return fail(err, "at most 8 inner slabs per outer slab");
    } else {
        P->tau_i = P->tau_o = p->levels[0].tau;
        P->n_i = p->levels[0].n_iter;
        P->k_i = p->levels[0].k_sweeps;
        P->n_o = 1;
        P->k_o = 0;
    }
    if (p->n_dirs < 1 || p->n_dirs > 3) return fail(err, "n_dirs must be 1..3");
    P->n_dirs = p->n_dirs;
    for (int i = 0; i < p->n_dirs; ++i) {
        if (p->dirs[i] < 0 || p->dirs[i] > 2) return fail(err, "charge axes must be 0, 1 or 2");
        for (int j = 0; j < i; ++j)
            if (p->dirs[j] == p->dirs[i]) return fail(err, "charge axes must be distinct");
        P->dirs[i] = p->dirs[i];
    }
    if (p->n_r < 1 || !p->r) return fail(err, "n_r must be >= 1 with a non-NULL r array");
    P->r.assign(p->r, p->r + p->n_r);
    if (p->n_probe < 0 || (p->n_probe > 0 && !p->probes)) return fail(err, "bad probe array");
    if (p->n_probe > 0) P->probes.assign(p->probes, p->probes + p->n_probe);
    if (p->n_comp < 0 || p->n_comp > 6 || (p->n_comp > 0 && !p->comps)) return fail(err, "n_comp must be 0..6");
    if (p->n_comp > 0) P->comps.assign(p->comps, p->comps + p->n_comp);
    for (int c : P->comps)
        if (c < 0 || c > 5) return fail(err, "components must be 0..5");
    if (P->probes.empty() != P->comps.empty()) return fail(err, "probes and components must both be given or both be empty");
    for (int e = 0; e < P->n_ens; ++e) {
        const u1ml_ensemble& E = P->ens[e];
        const int ext[4] = {E.ns[0], E.ns[1], E.ns[2], E.nt};
        for (int k = 0; k < 4; ++k)
            if (ext[k] < 2 || ext[k] % 2 != 0) return fail(err, "every extent must be even and >= 2 (ensemble " + std::to_string(e) + ")");
        if (!std::isfinite(E.beta) || E.beta < 0) return fail(err, "beta must be finite and >= 0");
        if (E.nt % P->tau_o != 0) return fail(err, "Nt must be a multiple of the outer tau");
        if (E.nt % P->tau_i != 0) return fail(err, "Nt must be a multiple of the inner tau");
        const double V = (double)E.ns[0] * E.ns[1] * E.ns[2] * E.nt;
        if (4.0 * V >= 4294967296.0) return fail(err, "4 V must fit in 32 bits (link ids)");
        // the kernels address an ensemble's links with 32-bit byte offsets
        if (4.0 * V * (P->precision == U1ML_FP64 ? 8 : 4) >= 4294967296.0)
            return fail(err, "the links of one ensemble (4 V words) must stay below 4 GiB");
        if ((double)E.ns[1] * E.ns[2] >= 4194304.0) return fail(err, "Ny * Nz must be below 2^22");
        if (E.nt >= 4194304) return fail(err, "Nt must be below 2^22");
        if ((double)E.ns[0] / 2 * E.ns[1] * E.ns[2] >= 16777216.0) return fail(err, "Ns^3 / 2 must be below 2^24");
        for (int i = 0; i < P->n_dirs; ++i) {
            const int d = P->dirs[i];
            for (int rv : P->r)
                if (rv < 1 || rv >= E.ns[d]) return fail(err, "every r must satisfy 1 <= r < Ns along the charge axis");
            for (const u1ml_probe& pr : P->probes) {
                const int n1 = E.ns[(d + 1) % 3], n2 = E.ns[(d + 2) % 3];
                if (std::abs(pr.p1) * 2 >= n1) return fail(err, "probe |p1| must be < Ns/2");
                if (std::abs(pr.p2) * 2 >= n2) return fail(err, "probe |p2| must be < Ns/2");
                if (std::abs(pr.l) >= E.ns[d]) return fail(err, "probe |l| must be < Ns along the charge axis");
                if (pr.mode != 0 && pr.mode != 1) return fail(err, "probe mode must be 0 or 1");
            }
        }
    }
    P->nd_cfg = 2ll * P->r.size() + 4ll * P->r.size() * P->probes.size() * P->comps.size() + 12 + P->r.size();
    if (p->form < U1ML_FORM_AUTO || p->form > U1ML_FORM_SPECTRAL) return fail(err, "form must be 0, 1 or 2");
    P->form_req = p->form;
    if (p->form == U1ML_FORM_SPECTRAL)
        for (const u1ml_ensemble& E : P->ens)
            for (int i = 0; i < P->n_dirs; ++i)
                if ((long long)E.ns[0] * E.ns[1] * E.ns[2] / E.ns[P->dirs[i]] > 4096)
                    return fail(err, "spectral form: a transverse plane has more than 4096 sites");
    // probes sharing (l, mode) share one longitudinal offset per (r, component)
    P->pgroup.clear();
    P->gdesc.clear();
    for (const u1ml_probe& pr : P->probes) {
        int g = 0;
        while (g < (int)P->gdesc.size() / 2 && !(P->gdesc[2 * g] == pr.l && P->gdesc[2 * g + 1] == pr.mode)) ++g;
        if (g == (int)P->gdesc.size() / 2) {
            P->gdesc.push_back(pr.l);
            P->gdesc.push_back(pr.mode);
        }
        P->pgroup.push_back(g);
    }
    // slot keys of the insertion contraction: the (probe, component) pairs
    // of each probe group whose plaquettes span the axis, then those whose
    // plaquettes do not (probes, then components, in problem order); blocks
    // of KS slots of one key, KS in {9, 6, 3, 1}, or kMfSlots for the
    // matrix-core kernel (the planner's choice, pack_slot_blocks)
    P->skeys.clear();
    P->skey_l.clear();
    P->skey_mode.clear();
    P->skey_spans.clear();
    for (int g = 0; g < (int)P->gdesc.size() / 2; ++g)
        for (int sp = 1; sp >= 0; --sp) {
            std::vector<std::pair<int, int>> slots;
            for (int p = 0; p < (int)P->probes.size(); ++p)
                if (P->pgroup[p] == g)
                    for (int ic = 0; ic < (int)P->comps.size(); ++ic)
                        if ((int)comp_spans_axis_host(P->comps[ic]) == sp) slots.emplace_back(p, ic);
            if (slots.empty()) continue;
            P->skeys.push_back(slots);
            P->skey_l.push_back(P->gdesc[2 * g]);
            P->skey_mode.push_back(P->gdesc[2 * g + 1]);
            P->skey_spans.push_back(sp);
        }
    // the block size whose padded work (slots rounded up to whole blocks,
    // separations to whole groups of ins_kr(KS)) is least; on a tie FP32 O
    // rows take the smaller block (each O value is converted to FP64 where it
    // is read, once per ins_kr(KS) separations: C2 FP32 11.51 ms per
    // configuration with blocks of 3 against 11.72 with 9) and FP64 rows the
    // larger (C2 FP64 16.80 ms with 9 against 17.05 with 3); blocks of 1 only
    // where they pad least (eight separations per work-item form more T)
    const size_t R_ = P->r.size();
    double best = 1e300;
    int best_ks = 1;
    const bool fp32_o = P->precision == U1ML_FP32;
    for (int ks : {9, 6, 3, 1}) {
        size_t padded = 0;
        for (const auto& k : P->skeys) padded += (k.size() + ks - 1) / ks * ks;
        const int kr = ins_kr(ks);
        const double work = (double)padded * (double)((R_ + kr - 1) / kr * kr);
        if (work < best || (fp32_o && work == best && ks >= 3)) {
            best = work;
            best_ks = ks;
        }
    }
    P->ins_ks_vec = best_ks;
    pack_slot_blocks(P, best_ks);
    return true;
}

// Bodies of more than kMaxGraphPhases are launched directly instead of through
// one captured graph, a phase counted also where sweeps take fewer launches: a
// single capture of a full configuration of the largest preset (about 275,000
// kernel nodes in one chain) ended the process with a segmentation fault, so
// graphs stay at the sizes that are tested; and a graph's first launch costs
// what its replays of so many launches gain back only after tens of them (300
// sweeps of 24^3 x 8, 5120 launches: 29.6 ms the first time and 19.1 then, launched
// directly 20.1 and 19.1).
constexpr long long kMaxGraphPhases = 8192;

long long body_phases(const Problem& P)
{
    const long long sweep = (1ll + P.n_or) * 8, meas = 1 + (P.multihit ? 1 : 0) + (P.spectral ? 6 : 0);
    const long long level = (long long)P.n_o * ((long long)P.k_o * sweep + (long long)P.n_i * (P.k_i * sweep + meas) + 6);
    return (P.spectral && P.two ? 2 : 1) * level + 10 + 5ll * P.n_ens;
}

// Kernel launches of one multilevel body (upper bound, of the whole batch on one
// lane), and
// of n sweeps of a class (0 full, 1 inner slabs, 2 outer slabs)
long long sweep_launches(const Problem& P, int cls, long long n)
{
    if (n == 0) return 0;
    if (P.slab_on[cls]) return (n + kSlabSweeps - 1) / kSlabSweeps;
    const int paired = (P.n_or + 1) / 2 * 2;  // passes with both-parities launches
    long long pass = 0;
    for (int mu = 0; mu < 4; ++mu) pass += P.pair_on[mu == 3 ? 9 : 3 * mu + cls] ? 1 : 2;
    return n * (paired * pass + (1 + P.n_or - paired) * 8);
}

long long body_launches(const Problem& P)
{
    const int outer = P.tau_o == P.tau_i ? 1 : 2;
    // per measurement: one (two with multihit); per inner level: the copies of frozen links (2), the two
    // contractions, the combine, the exponent pass (2) and the weights; in the spectral form, once per
    // measurement, staging, plane transforms and spectral sums (in parts past kMaxGrid work-groups)
    double tiles = 0.0;
    for (const u1ml_ensemble& E : P.ens) {
        const double nsig = (double)E.ns[0] * E.ns[1] * E.ns[2];
        double plane = 0.0;
        for (int i = 0; i < P.n_dirs; ++i) plane = std::max(plane, nsig / E.ns[P.dirs[i]]);
        tiles += (double)P.n_dirs * (E.nt / P.tau_i) * (double)(P.gdesc.size() / 2) * std::ceil(plane / kMacK);
    }
    const long long spectral = 3 + (long long)(tiles / kMaxGrid);
    const long long meas = 1 + (P.multihit ? 1 : 0);
    const long long level = (long long)P.n_o * ((P.two ? sweep_launches(P, outer, P.k_o) : 0) +
                                                (long long)P.n_i * (sweep_launches(P, 1, P.k_i) + meas) + 8);
    const long long passes = (P.spectral && P.two) ? 2 : 1;
    // per configuration: products (4), vacuum, spectral final (2), outer
    // weights, ring and counters; per ensemble: up to three fills and two
    // link copies
    return passes * level + (P.spectral ? spectral * P.n_o * P.n_i : 0) + 10 + 5ll * P.n_ens;
}

// probe groups of the slab-product launch: every probe in the history form,
// one (the correlator only) otherwise; the work-group table, the partial
// buffer and the launch all use this count
int prod_groups(const Problem& P) { return (!P.spectral && !P.probes.empty()) ? (int)P.probes.size() : 1; }

// --- both-parities launches (k_pair.hip) ----------------------------------
// Core rows along one axis k (y, z, t) of a class: its extent, whether the
// halo applies (not along mu, not across frozen layers, not where the tile is
// the whole extent).
struct PairGeo {
    int mu, nxh, N[3], slabs;
    int ext[3];  // lattice extents along y, z, t
    bool masked;
    bool halo(int k, int L) const { return k + 1 != mu && !(masked && k == 2) && L < N[k]; }
    PairGeo(const u1ml_ensemble& E, int cls, int tau)
        : mu(cls == 9 ? 3 : cls / 3), nxh(E.ns[0] / 2), slabs(tau > 1 ? E.nt / tau : 1), masked(tau > 1)
    {
        N[0] = E.ns[1];
        N[1] = E.ns[2];
        N[2] = masked ? tau - 1 : E.nt;
        ext[0] = N[0];
        ext[1] = N[1];
        ext[2] = E.nt;
    }
    int rows(const int* L) const  // of a tile, with its halo
    {
        const int core = L[0] * L[1] * L[2];
        int n = core;
        for (int k = 0; k < 3; ++k)
            if (halo(k, L[k])) n += 2 * (core / L[k]);
        return n;
    }
    // what a tile's rows depend on: direction, lattice, core, and how far (up
    // to the two steps its rows reach) the core lies from the lattice's ends
    std::array<int, 15> shape(const int* o, const int* L) const
    {
        std::array<int, 15> key = {mu, masked, nxh};
        for (int k = 0; k < 3; ++k) {
            const int v[4] = {ext[k], L[k], std::min(o[k], 2), std::min(ext[k] - o[k] - L[k], 2)};
            std::copy(v, v + 4, &key[3 + 4 * k]);
        }
        return key;
    }
};

// The tile with the least time per SIMD: a work-group's waves run on one of 256
// compute units (4 SIMDs each), so a unit holds its share of whole work-groups
// (share: this ensemble's part of the batch); halo rows are updated once more
// for every tile they touch.  24^3 x 8, temporal links: 3 x 3 rows (512
// work-groups, two per unit, of 4 waves) 84.4 us a sweep, 4 x 4 (288, on some
// units two, of 6 waves) 87.0, 6 x 6 87.7.
PairTile pair_tile(const PairGeo& G, double share, int max_threads, double* waves)
{
    PairTile best;
    double best_cost = 1e300;
    const int cap = max_threads / G.nxh, lt0 = G.masked ? G.N[2] : 1;  // rows of a work-group
    for (int ly = 1; ly <= std::min({G.N[0], 64, cap}); ++ly)
        for (int lz = 1; lz <= std::min({G.N[1], 64, cap / ly}); ++lz)
            for (int lt = lt0; lt <= std::min({G.N[2], 64, cap / (ly * lz)}); ++lt) {
                const int L[3] = {ly, lz, lt};
                if (G.rows(L) > cap) continue;
                long long tiles = G.slabs;
                for (int k = 0; k < 3; ++k) tiles *= (G.N[k] + L[k] - 1) / L[k];
                const int core = ly * lz * lt, rows = G.rows(L);
                const double w1 = (double)((rows * G.nxh + 63) / 64), w2 = (double)((core * G.nxh + 63) / 64);
                const double lat = std::ceil((double)tiles / share / 256) * std::max(1.0, w1 / 4);
                const double thr = (double)tiles / share * (w1 + w2) / 2 / 1024;
                const double cost = std::max(lat, thr) + 0.1 * thr;
                if (cost < best_cost) {
                    best_cost = cost;
                    std::copy(L, L + 3, best.L);
                    best.blocks = tiles;
                    *waves = (double)tiles * (w1 + w2) / 2;
                }
            }
    return best;
}

// The rows of the tile with origin o (y, z, t) and core L.
void pair_rows(const PairGeo& G, int word, const int* o, const int* L, PairRow* rows)
{
    int halo[3], n = L[0] * L[1] * L[2];  // first halo row of axis k: the faces below, then the faces above
    for (int k = 0; k < 3; ++k) {
        halo[k] = n;
        if (G.halo(k, L[k])) n += 2 * (L[0] * L[1] * L[2] / L[k]);
    }
    auto core = [&](const int* i) { return i[0] + L[0] * (i[1] + L[1] * i[2]); };
    auto face = [&](int k, int up, const int* i) {
        const int a = (k + 1) % 3, b = (k + 2) % 3;
        return halo[k] + up * (L[a] * L[b]) + i[a] + L[a] * i[b];
    };
    // byte offset from the origin of the row displaced by d, and one step further along axis k
    auto offset = [&](const int* d, int k, int step) {
        int c[3];
        for (int a = 0; a < 3; ++a) {  // at most two steps past either end, extents are at least 2
            const int x = o[a] + d[a] + (a == k ? step : 0);
            c[a] = (x < 0 ? x + G.ext[a] : x >= G.ext[a] ? x - G.ext[a] : x) - o[a];
        }
        return word * G.nxh * (c[0] + G.ext[0] * (c[1] + G.ext[1] * c[2]));
    };
    auto fill = [&](PairRow* r, const int* d) {
        r->c = offset(d, 0, 0);
        r->p1 = offset(d, 0, 1), r->m1 = offset(d, 0, -1);
        r->p2 = offset(d, 1, 1), r->m2 = offset(d, 1, -1);
        r->p3 = offset(d, 2, 1), r->m3 = offset(d, 2, -1);
        r->par = (d[0] + d[1] + d[2]) & 1;
    };
    int i[3];
    for (i[2] = 0; i[2] < L[2]; ++i[2])
        for (i[1] = 0; i[1] < L[1]; ++i[1])
            for (i[0] = 0; i[0] < L[0]; ++i[0]) {
                PairRow* r = &rows[core(i)];
                fill(r, i);
                unsigned* lds[3] = {&r->ly, &r->lz, &r->lt};
                for (int k = 0; k < 3; ++k) {
                    if (k + 1 == G.mu) continue;
                    unsigned code[2];
                    for (int up = 0; up < 2; ++up) {
                        int j[3] = {i[0], i[1], i[2]};
                        j[k] += up ? 1 : -1;
                        int id;
                        if (j[k] >= 0 && j[k] < L[k]) {
                            id = core(j);
                        } else if (G.masked && k == 2) {
                            id = -1;
                        } else if (!G.halo(k, L[k])) {
                            j[k] = up ? 0 : L[k] - 1;
                            id = core(j);
                        } else {
                            id = face(k, up, i);
                            fill(&rows[id], j);
                        }
                        code[up] = id < 0 ? kPairFrozen : (unsigned)(id * G.nxh * word);
                    }
                    *lds[k] = code[1] << 16 | code[0];
                }
            }
}

// Every tile of ensemble k in class cls: f(origin, core extents), time
// fastest (the tiles of one stretch of the slices at consecutive times follow
// each other).
template <typename F>
void pair_for_tiles(const Problem& P, int cls, int k, F f)
{
    const int tau = P.pair_tau(cls);
    const PairGeo G(P.ens[k], cls, tau);
    const PairTile& T = P.pair_tile[cls][k];
    for (int z = 0; z < G.N[1]; z += T.L[1])
        for (int y = 0; y < G.N[0]; y += T.L[0])
            for (int s = 0; s < G.slabs; ++s)
                for (int t = 0; t < G.N[2]; t += T.L[2]) {
                    const int L[3] = {std::min(T.L[0], G.N[0] - y), std::min(T.L[1], G.N[1] - z),
                                      std::min(T.L[2], G.N[2] - t)};
                    const int o[3] = {y, z, G.masked ? s * tau + 1 : t};
                    f(o, L);
                }
}

// Chooses, per class of sweeps (full, inner slabs, outer slabs), whether sweeps
// run in LDS, one work-group per slab or lattice: where a phase of every
// ensemble's slab has at most one link per work-item of a work-group and its
// links fit LDS.  MI355X, us per sweep otherwise / in LDS: FP32 4^4 full 48 / 27,
// 8^3 x 4 (1024 links a phase) 59 / 52, 10^3 x 4 (2000) 69 / 97; slabs of 2 with a
// measurement each, 8^3 (512) 55 / 45, 10^3 (1000) 65 / 59, 12^3 (1728) 63 / 83;
// FP64 4^4 full 80 / 52, 6^3 x 4 (432) 94 / 83, 8^3 x 4 (1024) 92 / 157; slabs of
// 8^3 (512) 90 / 78, 10^3 (1000) 99 / 121.
// Not for batches that fill the device either way, where a launch per direction
// hides more latency than work-groups that stand at their barriers, and no wave
// idles for a slab that does not fill it.  us per sweep otherwise / in LDS, FP64
// (whose compute units hold 16 of these waves): slabs of 8^3 512 / 768 / 1024 of
// them 151 / 184 / 223, 124 / 185 / 245; 1024 / 2048 of 6^3 152 / 219, 136 / 258; full
// 6^3 x 4, 768 / 1024 lattices 280 / 306, 240 / 323; 4096 / 8192 slabs of 2 x 4 x 4
// 137 / 176, 138 / 259; rows of at most 2 half sites are slow otherwise: 8192 / 32768
// slabs of 4^3 204 / 518, 144 / 513.  FP32 full 8 x 8 x 16 x 2, 1536 / 3072 lattices 333 /
// 578, 311 / 617; 8192 / 16384 slabs of 2 x 4 x 4 96 / 137, 89 / 164.
void plan_slabs(Problem* P)
{
    const int word = P->precision == U1ML_FP64 ? 8 : 4;
    const int max_threads = P->precision == U1ML_FP64 ? kSlabThreads<double> : kSlabThreads<float>;
    const bool hb = P->update == U1ML_UPDATE_HEATBATH;
    for (int cls = 0; cls < 3; ++cls) {
        const int tau = cls == 0 ? 0 : (cls == 1 ? P->tau_i : P->tau_o);
        bool ok = cls != 2 || P->two;
        size_t lds = 0, blocks = 0;
        int threads = 64, nxh = 1;
        double links_all = 0.0;  // of the largest phase, every work-group
        for (const u1ml_ensemble& E : P->ens) {
            const double links = (double)E.ns[0] / 2 * E.ns[1] * E.ns[2] * (tau ? tau : E.nt);  // of the largest phase
            ok = ok && links <= max_threads;
            if (ok) threads = std::max(threads, ((int)links + 63) / 64 * 64);
            blocks += tau ? E.nt / tau : 1;
            links_all += links * (tau ? E.nt / tau : 1);
            nxh = std::max(nxh, E.ns[0] / 2);
        }
        for (const u1ml_ensemble& E : P->ens)
            if (ok)
                lds = std::max(lds, slab_lds(E.ns[0] / 2 * E.ns[1] * E.ns[2], tau ? tau + 1 : E.nt, threads, hb, word));
        const int wg = threads / 64;
        const double waves = (double)blocks * wg, filled = links_all / 64;
        const double held = waves * 16 / (16 / wg * wg);  // waves and the places that they leave empty
        const bool few = P->precision == U1ML_FP64
                             ? held <= (held > 4 * filled ? 1024 : 6144) || (held <= 1.1 * filled && nxh <= 2)
                             : (cls == 0 && threads > 768 ? waves <= 24576 : waves <= 8192 || waves <= 1.9 * filled);
        P->slab_on[cls] = ok && lds <= kSlabLds && few;
        P->slab_block[cls] = threads;
        P->slab_lds_bytes[cls] = P->slab_on[cls] ? lds : 0;
        P->slab_blocks[cls] = P->slab_on[cls] ? blocks : 0;
    }
}

// Chooses, per class, whether sweeps update both parities in one launch, and
// the tiles.  What a direction gains (us; negative: one launch is faster) as
// fitted to 84 lattices and batches of 6^3 x 64 to 32 x 16^3 x 4, every direction
// with and without, root-mean-square error 0.8 (FP64 1.2) of a spread of 1.4
// (2.6): a launch saved, against waves that hold more and so hide less of each
// other's latency (FP64 above all: past one wave per SIMD an added one costs
// what it costs in two launches), halo waves, and runs of the tile in memory
// shorter than a few cache lines, whose lines are fetched for their neighbours
// as well.  MI355X, us per sweep with none / with this rule, full: FP32 24^3 x 8
// 89.1 / 78.2, 12^3 x 96 99.8 / 96.1 (113 with every direction paired), 32 of
// 12^3 x 8 112.9 / 107.6 (158); FP64 8^3 x 512 147.8 / 142.6 (208), 24^3 x 12 149.1 /
// 148.9 (215); inside slabs: FP32 24^3 x 8 84.7 / 62.8, FP64 117.8 / 101.0, 24^3 x 24
// 160.7 / 157.3 (175).  None of 118 lattices and batches loses more than 2 %.
struct PairFit {
    double fixed, one, two, lines, halo;
    double most;  // paired below this
};
constexpr PairFit kPairFit[2] = {{-1.09, 2.85, -2.78, 1.11, 0.66, -0.3}, {-1.31, 0.54, -0.44, 0.51, 0.33, 0.2}};  // FP64, FP32
constexpr double kPairWaves = 4.2;  // waves per SIMD that the fit reaches

double pair_gain(int precision, double one, double two, double lines)
{
    const PairFit& f = kPairFit[precision];
    return f.fixed + f.one * std::max(1.0, one) + f.two * std::max(1.0, two) + f.lines * lines + f.halo * std::max(0.0, one - two);
}

void plan_pairs(Problem* P)
{
    double vol = 0.0;
    size_t bytes = 0;
    const size_t word = P->precision == U1ML_FP64 ? 8 : 4;
    std::map<std::array<int, 4>, int> first;
    P->lattice.clear();
    for (int k = 0; k < P->n_ens; ++k) {
        const u1ml_ensemble& E = P->ens[k];
        const double v = (double)E.ns[0] * E.ns[1] * E.ns[2] * E.nt;
        vol += v;
        bytes += (size_t)(4.0 * v) * word;
        P->lattice.push_back(first.emplace(std::array<int, 4>{E.ns[0], E.ns[1], E.ns[2], E.nt}, k).first->second);
    }
    const int max_threads = P->precision == U1ML_FP64 ? kPairThreads<double> : kPairThreads<float>;
    for (int cls = 0; cls < kPairClasses; ++cls) {
        P->pair_on[cls] = false;
        P->pair_tile[cls].assign(P->n_ens, PairTile());
        const int tau = P->pair_tau(cls);
        // both buffers of an ensemble within 32-bit offsets of its links; not for sweeps in LDS, nor where a
        // sweep is one pass (which ends in the first buffer, see enq_sweep)
        bool ok = 2 * bytes < 4294967296.0 && (cls % 3 != 2 || P->two) && P->n_or > 0;
        if (cls < 9) ok = ok && !P->slab_on[cls % 3];
        else ok = ok && !(P->slab_on[0] && P->slab_on[1] && (!P->two || P->slab_on[2]));
        // waves of either form; least: of one launch without halo; lines: waves over 64-byte lines of a run
        double one = 0.0, two = 0.0, least = 0.0, lines = 0.0;
        for (const u1ml_ensemble& E : P->ens) {
            const PairGeo G(E, cls, tau);
            const double slice = (double)G.nxh * G.N[0] * G.N[1];
            two += std::ceil(slice / 64) * G.N[2] * G.slabs;
            least += slice / 64 * G.N[2] * G.slabs;
        }
        // no tiles to look for where the gain without any halo is not enough
        ok = ok && least < kPairWaves * 1024 && pair_gain(P->precision, least / 1024, two / 1024, 0.0) < 0.8;
        P->pair_block[cls] = 64;
        std::vector<double> waves(ok ? P->n_ens : 0), run(waves);
        for (int k = 0; ok && k < P->n_ens; ++k) {
            const int l = P->lattice[k];  // equal lattices have equal tiles
            if (l == k) {
                const u1ml_ensemble& E = P->ens[k];
                const PairGeo G(E, cls, tau);
                const double v = (double)E.ns[0] * E.ns[1] * E.ns[2] * E.nt;
                const PairTile T = pair_tile(G, v / vol, max_threads, &waves[k]);
                ok = T.blocks > 0;
                P->pair_tile[cls][k] = T;
                run[k] = (double)G.nxh * word * T.L[0];  // bytes of the tile in one piece
                for (int a = 1; a < 3 && T.L[a - 1] == G.ext[a - 1]; ++a) run[k] *= T.L[a];
                if (ok) P->pair_block[cls] = std::max(P->pair_block[cls], (G.rows(T.L) * G.nxh + 63) / 64 * 64);
            } else {
                P->pair_tile[cls][k] = P->pair_tile[cls][l];
                waves[k] = waves[l];
                run[k] = run[l];
            }
            one += waves[k];
            if (run[k] < 512) lines += waves[k] * 64 / run[k];
        }
        // where the fit is too high in FP64: below 0.8 waves per SIMD (by up to 0.9 us), and for temporal links,
        // whose tiles lie in one slice, up to 1.5 (by 0.3 to 0.8 us)
        double most = kPairFit[P->precision].most;
        if (one < 0.8 * 1024) most = std::max(most, 0.0);
        if (cls == 9 && one < 1.5 * 1024) most = std::max(most, 0.8);
        // (and too low by up to 1.4 us, as often as it is right, for temporal tiles with a halo past 2.2)
        ok = ok && !(cls == 9 && one > 2.2 * 1024 && one > 1.1 * two);
        P->pair_on[cls] = ok && one < kPairWaves * 1024 &&
                          pair_gain(P->precision, one / 1024, two / 1024, lines / 1024) < most;
    }
    P->n_pair_rows = 0;
    P->pair_shape.clear();
    for (int cls = 0; cls < kPairClasses; ++cls)
        for (int k = 0; P->pair_on[cls] && k < P->n_ens; ++k) {
            if (P->lattice[k] != k) continue;  // the rows of an equal lattice
            const PairGeo G(P->ens[k], cls, P->pair_tau(cls));
            pair_for_tiles(*P, cls, k, [&](const int* o, const int* L) {
                if (P->pair_shape.try_emplace(G.shape(o, L), P->n_pair_rows).second) P->n_pair_rows += G.rows(L);
            });
        }
}

// the row table of the shapes that plan_pairs found
std::vector<PairRow> build_pair_rows(const Problem& P)
{
    std::vector<PairRow> rows(P.n_pair_rows, PairRow{});
    const int word = P.precision == U1ML_FP64 ? 8 : 4;
    int next = 0;  // shapes come in the order of their first rows
    for (int cls = 0; cls < kPairClasses; ++cls)
        for (int k = 0; P.pair_on[cls] && k < P.n_ens; ++k) {
            if (P.lattice[k] != k) continue;
            const PairGeo G(P.ens[k], cls, P.pair_tau(cls));
            pair_for_tiles(P, cls, k, [&](const int* o, const int* L) {
                if (P.pair_shape.at(G.shape(o, L)) != next) return;
                pair_rows(G, word, o, L, &rows[next]);
                next += G.rows(L);
            });
        }
    return rows;
}

// History form, vector kernel: slot blocks per work-group of an ensemble whose
// longest line has nmax sites, and measurements per LDS chunk buffer (static
// LDS of the kernel): fewer slot blocks while a chunk would hold fewer than 8
// measurements, or not even one.  False where one does not fit at all.
bool ins_shape(const Problem& P, int ks, int nsb, int nmax, int* pbw, int* mc)
{
    const int kr = ins_kr(ks), word = P.precision == U1ML_FP64 ? 8 : 4;
    const int unit = nmax * (((int)P.r.size() + kr - 1) / kr);  // tasks of one slot block
    int b = std::max(1, std::min(std::min(nsb, kInsThreads / unit), kInsRowsMax / (2 * ks)));
    auto fit_mc = [&](int bpw) {
        int m = std::min(P.n_i, kInsPh);
        while (m > 1 && !ins_chunk_fits(m, nmax, bpw * ks * 2, word)) --m;
        return m;
    };
    while (b > 1 && (!ins_chunk_fits(1, nmax, b * ks * 2, word) || fit_mc(b) < std::min(8, P.n_i))) --b;
    *pbw = b;
    *mc = fit_mc(b);
    return ins_chunk_fits(*mc, nmax, b * ks * 2, word);
}

bool compute_sizes(Problem& P, Sizes* S, u1ml_plan_info* info, Layout* Lo, std::string* err)
{
    const size_t word = P.precision == U1ML_FP64 ? 8 : 4;
    const bool store_o = !P.probes.empty();
    const size_t R = P.r.size(), Np = P.probes.size(), Nc = P.comps.size(), nd = (size_t)P.n_dirs;
    const size_t NG = P.gdesc.size() / 2;
    // contraction form: the spectral form needs every transverse plane of a
    // charge axis within 4096 sites.  AUTO estimates the device time each
    // form adds to a configuration and takes the smaller (history also when
    // the spectral form does not apply, spectral when the history form's
    // per-site averages would exceed 64 GiB).  Fits to 260 random problems on
    // MI355X (both link types, 6^3 to 48^3 and unequal extents, 1 to 64
    // ensembles, 1 to 105 probes, one and two levels; 20 to 35 % rms):
    //   history:  18 ns per work-group of the insertion sums and 9 ns per LDS
    //             chunk of measurements (they overlap; the products run
    //             beside them), O rows of lines that are not contiguous
    //             staged at 1 TB/s, averages read back at 3.3 TB/s; two
    //             levels: 50 us per outer update, averages written and folded
    //             into the outer sums at 5.5 TB/s;
    //   spectral: per measurement 15 us of dependent launches, 9.5 ps per
    //             plane element and field (staging and transforms; planes
    //             that the transforms in registers do not take 30 ps and 8 ns
    //             per plane more), spectra and running sums read for the
    //             spectral sums at 4.1 TB/s; two levels: the replay repeats
    //             every update (FP32 9e10 link updates/s and 13 us per pass
    //             over the lattice, FP64 4.3e10 and 21 us).
    // On those problems the choice costs 0.2 % of the better form's time, 1.17
    // times in the worst; with history at 6.6e12 FMA/s alone and 0.198 ps per
    // flop of the spectral sums, fitted to earlier kernels, it cost 13 %, up to
    // 5.7 times.
    // Measured per configuration (history / spectral, ms): 24^3x8, 9 probes,
    // 100 updates 8.2 / 10.0; 24^3x8 in-plane map 13.1 / 13.0; 48^3x12 two
    // levels 2 x 10, 1 probe 8.5 / 14.2, 8 probes 37.9 / 14.2.
    // The history form's kernel: matrix cores where 0.18 of the FP64 matrix
    // peak per 16 x 16 x 4 step, padding included, is less than 6.6e12 FMA/s
    // of the vector kernel (3.3 ms per launch on 24^3x8 with 9 probes against
    // 1.5; a plain stream of these steps runs at 46 TFLOP/s, FP64 vector FMA
    // at 61); that rate covers the averages' traffic, too.
    {
        bool plane_ok = true, hist_fits = true;
        double hist_avg = 0.0, est_h = 0.0, est_s = 0.0, est_ins = 0.0, est_rd = 0.0, est_v = 0.0, est_m = 0.0;
        const double n_lev = P.two ? P.n_o : 1, n_meas = (double)P.n_i * n_lev;
        const double n_steps = (double)((P.n_i + 3) / 4) * n_lev;  // MFMA steps of 4 measurements
        const int ks = P.ins_ks_vec;
        size_t nblk8 = 0, nsb = 0;
        for (const auto& k : P.skeys) {
            nblk8 += (k.size() + kMfSlots - 1) / kMfSlots;
            nsb += (k.size() + ks - 1) / ks;
        }
        const int word_o = (int)word;
        bool mf_ok = R <= (size_t)kMfR;
        int side = -1, npm = 0;  // side of every plane if all are squares of one side, else 0; largest extent
        for (const u1ml_ensemble& E : P.ens)
            for (int i = 0; i < P.n_dirs; ++i)
                for (int k = 1; k < 3; ++k) {
                    const int len = E.ns[(P.dirs[i] + k) % 3];
                    if (side < 0) side = len;
                    if (side != len) side = 0;
                }
        const bool fast = fft_in_registers(side);
        double upd = 0.0;
        for (const u1ml_ensemble& E : P.ens) {
            const double nsig = (double)E.ns[0] * E.ns[1] * E.ns[2];
            double lines = 0.0, planes = 0.0, strided = 0.0;  // lines of the axes; their planes; axes with strided lines
            for (int i = 0; i < P.n_dirs; ++i) {
                const int len = E.ns[P.dirs[i]];
                if (nsig / len > 4096.0) plane_ok = false;
                lines += nsig / len;
                planes += len;
                strided += P.dirs[i] != 0 || len * word % 16 != 0 ? 1.0 : 0.0;
            }
            const int nmax = std::max(E.ns[0], std::max(E.ns[1], E.ns[2]));  // as the contraction is sized
            npm = std::max(npm, nmax);
            if (!mf_chunk_fits(4, nmax, (int)R, 2 * kMfSlots, word_o)) mf_ok = false;
            const double per = (double)nd * R * Np * Nc * 2 * nsig * 16.0;
            const double si = (double)(E.nt / P.tau_i), so = P.two ? (double)(E.nt / P.tau_o) : 0.0;
            hist_avg += per * si + per * so;
            est_v += n_meas * nd * si * nsig * R * Np * Nc * 4.0 / 6.6e12;
            est_m += n_steps * nd * si * nsig * (double)((R + 7) / 8) * nblk8 * 1024.0 / (0.18 * 39.3e12);
            int pbw = 1, mc = 1;
            if (Np && !ins_shape(P, ks, (int)nsb, nmax, &pbw, &mc)) hist_fits = false;
            const double wgs = si * lines * (double)((nsb + pbw - 1) / pbw) * n_lev;
            est_ins += wgs * (18e-9 + (double)((P.n_i + mc - 1) / mc) * 9e-9) +
                       strided * n_meas * si * nsig * (double)nsb * ks * 2 * (double)word / 1.0e12;
            est_rd += per * (P.two ? so : si) / 3.3e12;
            if (P.two) est_h += n_lev * per * (si + 2 * so) / 5.5e12;
            const double el = si * nsig * (R + 12);  // plane elements of one axis
            const double run = si * R * Nc * 2 * (double)NG * lines * 16.0;  // the running sums, bytes
            est_s += n_meas * (nd * el * (fast ? 9.5e-12 : 40e-12) + (fast ? 0.0 : si * planes * (R + 12) * 8e-9) +
                               (nd * el * (double)NG * 16.0 + 2 * run) / 4.1e12);
            if (P.two) {
                const double V = nsig * E.nt, vh = V / 2;
                const double sp_i = vh / E.nt * (E.nt - si), sp_o = vh / E.nt * (E.nt - so);
                upd += n_lev * (1 + P.n_or) * 2 * ((double)P.k_o * (vh + 3 * sp_o) + (double)P.n_i * P.k_i * (vh + 3 * sp_i));
            }
        }
        est_s += n_meas * 15e-6;
        if (P.two) {
            est_h += n_lev * 50e-6;
            est_s += upd / (P.precision == U1ML_FP64 ? 4.3e10 : 9e10) +
                     n_lev * ((double)P.k_o + (double)P.n_i * P.k_i) * (1 + P.n_or) *
                         (P.precision == U1ML_FP64 ? 21e-6 : 13e-6);
        }
        P.ins_mfma_est = Np && (P.ins_kernel == 2 || (P.ins_kernel == 0 && mf_ok && est_m < est_v));
        est_h += P.ins_mfma_est ? est_m : est_ins + est_rd;
        P.est_hist_ms = Np ? est_h * 1e3 : 0.0;
        P.est_spec_ms = (Np && plane_ok) ? est_s * 1e3 : -1.0;
        if (P.form_req == U1ML_FORM_SPECTRAL) {
            P.spectral = !P.probes.empty();  // planes checked by read_problem
        } else if (P.form_req == U1ML_FORM_AUTO) {
            // no form whose LDS does not hold the problem (spectral: extents above 106) where the other's does
            if (P.ins_mfma_est) hist_fits = true;
            const bool spec_fits = 2 * spec_mac_lds(npm) <= kSlabLds;
            P.spectral = !P.probes.empty() && plane_ok &&
                         (hist_avg > 64.0 * 1024 * 1024 * 1024 || (spec_fits && (est_s < est_h || !hist_fits)));
        } else {
            P.spectral = false;
        }
    }
    // slot blocks for the kernel that sums the history form
    if (Np && !P.spectral) {
        const int ks = P.ins_mfma_est ? kMfSlots : P.ins_ks_vec;
        if (P.ins_ks != ks) pack_slot_blocks(&P, ks);
    }
    plan_slabs(&P);
    plan_pairs(&P);
    const bool spec = P.spectral;
    size_t L = 0, HC = 0, HO = 0, AT = 0, ATO = 0, OT = 0, OTO = 0, VAC = 0, PP = 0, HIT = 0;
    size_t maxV = 0, paper = 0, upd_cfg = 0, upd_sweep = 0, blocks64 = 0, mblocks = 0;
    S->links.clear();
    S->hc.clear();
    S->ho.clear();
    S->at.clear();
    S->ato.clear();
    S->ot.clear();
    S->oto.clear();
    S->vac.clear();
    S->hit.clear();
    S->wf.clear();
    S->gf.clear();
    S->sph.clear();
    S->spo.clear();
    S->facc.clear();
    S->cpl.clear();
    S->opl.clear();
    size_t WF = 0, GF = 0, SPH = 0, SPO = 0, FACC = 0, CPL = 0, OPL = 0;
    for (const u1ml_ensemble& E : P.ens) {
        const size_t nsig = (size_t)E.ns[0] * E.ns[1] * E.ns[2];
        const size_t V = nsig * E.nt;
        maxV = std::max(maxV, V);
        blocks64 += (nsig / 2 + 63) / 64 * E.nt;  // update work-groups lie in one time slice
        blocks64 += 8;                            // padding of the XCD-aware block order
        const size_t si = E.nt / P.tau_i, so = E.nt / P.tau_o;
        size_t v, t;
        // links: 4 V words, padded to 256 bytes
        if (!mul_ok(4 * V, word, &v)) return fail(err, "size overflow (links)");
        S->links.push_back(L / word);
        L = align_up(L + v);
        S->hc.push_back(HC);
        // plain slab phases, then (multihit) the multihit ones
        if (!mul_ok((size_t)P.n_i * si * (P.multihit ? 2 : 1), nsig, &t) || !add_ok(HC, t, &HC))
            return fail(err, "size overflow (history)");
        HC = align_up(HC * 16) / 16;
        S->ho.push_back(HO);
        if (store_o) {
            if (!mul_ok((size_t)P.n_i * si * 12, nsig, &t) || !add_ok(HO, t, &HO)) return fail(err, "size overflow (history)");
            HO = align_up(HO * word) / word;
        }
        S->at.push_back(AT);
        AT = align_up((AT + nd * R * si * nsig) * 16) / 16;
        S->ato.push_back(ATO);
        if (store_o && !spec) {
            if (!mul_ok(nd * R * Np * Nc * 2 * si, nsig, &t) || !add_ok(ATO, t, &ATO)) return fail(err, "size overflow (averages)");
            ATO = align_up(ATO * 16) / 16;
        }
        S->ot.push_back(OT);
        S->oto.push_back(OTO);
        if (P.two) {
            OT = align_up((OT + nd * R * so * nsig) * 16) / 16;
            if (store_o && !spec) {
                if (!mul_ok(nd * R * Np * Nc * 2 * so, nsig, &t) || !add_ok(OTO, t, &OTO)) return fail(err, "size overflow (outer)");
                OTO = align_up(OTO * 16) / 16;
            }
        }
        S->wf.push_back(WF);
        S->gf.push_back(GF);
        S->sph.push_back(SPH);
        S->spo.push_back(SPO);
        S->facc.push_back(FACC);
        S->cpl.push_back(CPL);
        S->opl.push_back(OPL);
        if (spec) {
            CPL = align_up((CPL + nd * si * nsig) * 16) / 16;
            OPL = align_up((OPL + nd * si * 12 * nsig) * word) / word;
            size_t n12max = 0;
            for (int i = 0; i < P.n_dirs; ++i) n12max = std::max(n12max, nsig / (size_t)E.ns[P.dirs[i]]);
            if (P.two) WF = align_up((WF + nd * R * so * nsig) * 16) / 16;
            GF = align_up((GF + nd * R * si * nsig) * 16) / 16;
            SPH = align_up((SPH + nd * si * R * nsig) * 16) / 16;
            SPO = align_up((SPO + nd * si * 12 * nsig) * 16) / 16;
            if (!mul_ok(nd * si * R * Nc * 2 * NG, n12max, &t) || !add_ok(FACC, t, &FACC))
                return fail(err, "size overflow (spectral sums)");
            FACC = align_up(FACC * 16) / 16;
        }
        S->vac.push_back(VAC);
        S->hit.push_back(HIT);
        if (P.multihit) HIT += V;
        // running double-double vacuum partials, one set of 12 per measurement block
        VAC += ((nsig * si + 255) / 256) * 24;
        // slab-product partials: per (r, probe group, site chunk) work-group
        PP += R * (size_t)prod_groups(P) * ((nd * nsig + kProdChunk - 1) / kProdChunk) * kProdQ * 2;
        mblocks += (nsig * si + 255) / 256;
        // the paper's running accumulators: 2 doubles per site and per point of
        // the transverse plane, per slab of the inner level (Sec. II.D)
        const size_t area = (size_t)E.ns[(P.dirs[0] + 1) % 3] * E.ns[(P.dirs[0] + 2) % 3];
        paper += 2 * 8 * V * area / P.tau_i;
        // link updates
        const size_t vh = V / 2;
        const size_t sp_i = vh / E.nt * (E.nt - E.nt / P.tau_i);  // spatial links of one parity, one direction
        const size_t sp_o = vh / E.nt * (E.nt - E.nt / P.tau_o);
        const size_t per_sweep_i = (1 + P.n_or) * 2 * (vh + 3 * sp_i);
        const size_t per_sweep_o = (1 + P.n_or) * 2 * (vh + 3 * sp_o);
        upd_cfg += (size_t)P.n_o * ((size_t)P.k_o * per_sweep_o + (size_t)P.n_i * P.k_i * per_sweep_i);
        upd_sweep += (1 + P.n_or) * 4 * V;
    }
    Lo->sz_links = align_up(L);
    Lo->sz_hc = align_up(HC * 16);
    Lo->sz_ho = align_up(HO * word);
    Lo->sz_at = align_up(AT * 16);
    Lo->sz_ato = align_up(ATO * 16);
    Lo->sz_ot = align_up(OT * 16);
    Lo->sz_oto = align_up(OTO * 16);
    Lo->sz_wf = align_up(WF * 16);
    Lo->sz_gf = align_up(GF * 16);
    Lo->sz_sph = align_up(SPH * 16);
    Lo->sz_spo = align_up(SPO * 16);
    Lo->sz_facc = align_up(FACC * 16);
    Lo->sz_cpl = align_up(CPL * 16);
    Lo->sz_opl = align_up(OPL * word);
    Lo->sz_saved = (spec && P.two) ? Lo->sz_links : 0;
    size_t res;
    if (!mul_ok((size_t)P.max_configs * P.n_ens, (size_t)P.nd_cfg * 8, &res)) return fail(err, "size overflow (results)");
    Lo->sz_res = align_up(res);
    // scratch
    size_t s = 0;
    auto take = [&](size_t bytes) {
        const size_t o = s;
        s = align_up(s + bytes);
        return o;
    };
    const int n = P.n_ens;
    Lo->s_ens = take(sizeof(EnsDesc) * n);
    Lo->s_obs = take(sizeof(ObsDesc));
    Lo->s_r = take(sizeof(int) * R);
    Lo->s_probe = take(sizeof(int) * 4 * std::max<size_t>(Np, 1));
    Lo->s_comp = take(sizeof(int) * std::max<size_t>(Nc, 1));
    Lo->n_bstart_tables = kNumTabs;
    Lo->s_bstart = take(sizeof(int) * (n + 1) * kNumTabs);
    Lo->s_upd = take(sizeof(uint32_t) * n);
    Lo->s_ring = take(sizeof(int) * 4);
    Lo->s_vpart = take(sizeof(double) * VAC);
    Lo->s_hit = take(sizeof(double2) * HIT);
    Lo->s_ppart = take(sizeof(double) * 6 * kPlaqBlocks * n);
    Lo->s_pout = take(sizeof(double) * 6 * n);
    Lo->s_count = take(sizeof(unsigned long long) * 2);
    Lo->s_stage = take(sizeof(double) * 4 * maxV);
    Lo->bmap_stride = blocks64;
    Lo->s_bmap = take(sizeof(UpdBlock) * kUpdateClasses * blocks64);
    Lo->s_mmap = take(sizeof(MeasBlock) * mblocks);
    Lo->s_prow = take(sizeof(PairRow) * P.n_pair_rows);
    size_t pair_bytes[kPairClasses] = {};
    for (int cls = 0; cls < kPairClasses; ++cls) {
        size_t blocks = kXcds;  // padding of the XCD-aware block order
        for (const PairTile& T : P.pair_tile[cls]) blocks += (size_t)T.blocks;
        pair_bytes[cls] = P.pair_on[cls] ? sizeof(PairBlock) * blocks : 0;
        Lo->s_pmap[cls] = take(pair_bytes[cls]);
    }
    for (int cls = 0; cls < 3; ++cls) Lo->s_smap[cls] = take(sizeof(SlabBlock) * P.slab_blocks[cls]);
    Lo->s_prodpart = take(sizeof(double) * PP);
    for (int l = 0; l < kMaxLanes; ++l) {
        Lo->s_lens[l] = take(sizeof(EnsDesc) * n);
        Lo->s_lbstart[l] = take(sizeof(int) * (n + 1) * kNumTabs);
        Lo->s_lbmap[l] = take(sizeof(UpdBlock) * kUpdateClasses * blocks64);
        Lo->s_lmmap[l] = take(sizeof(MeasBlock) * mblocks);
        Lo->s_lring[l] = take(sizeof(int) * 4);
        for (int cls = 0; cls < kPairClasses; ++cls) Lo->s_lpmap[l][cls] = take(pair_bytes[cls]);
        for (int cls = 0; cls < 3; ++cls) Lo->s_lsmap[l][cls] = take(sizeof(SlabBlock) * P.slab_blocks[cls]);
    }
    Lo->s_pgroup = take(sizeof(int) * std::max<size_t>(Np, 1));
    Lo->s_gdesc = take(sizeof(int) * std::max<size_t>(2 * NG, 2));
    Lo->s_pblk = take(sizeof(int) * std::max<size_t>(P.pblk.size(), kInsBlkInts));
    Lo->sz_scr = s;
    size_t off = 0;
    Lo->off_links = off;
    off += Lo->sz_links;
    Lo->off_alt = off;
    if (P.any_pair()) off += Lo->sz_links;
    Lo->off_hc = off;
    off += Lo->sz_hc;
    Lo->off_ho = off;
    off += Lo->sz_ho;
    Lo->off_at = off;
    off += Lo->sz_at;
    Lo->off_ato = off;
    off += Lo->sz_ato;
    Lo->off_ot = off;
    off += Lo->sz_ot;
    Lo->off_oto = off;
    off += Lo->sz_oto;
    Lo->off_res = off;
    off += Lo->sz_res;
    Lo->off_wf = off;
    off += Lo->sz_wf;
    Lo->off_gf = off;
    off += Lo->sz_gf;
    Lo->off_sph = off;
    off += Lo->sz_sph;
    Lo->off_spo = off;
    off += Lo->sz_spo;
    Lo->off_facc = off;
    off += Lo->sz_facc;
    Lo->off_saved = off;
    off += Lo->sz_saved;
    Lo->off_cpl = off;
    off += Lo->sz_cpl;
    Lo->off_opl = off;
    off += Lo->sz_opl;
    Lo->off_scr = off;
    off += Lo->sz_scr;
    if (info) {
        std::memset(info, 0, sizeof(*info));
        info->ws_bytes = off;
        info->link_bytes = Lo->sz_links;
        info->history_bytes = Lo->sz_hc + Lo->sz_ho;
        info->average_bytes = Lo->sz_at + Lo->sz_ato;
        info->outer_bytes = Lo->sz_ot + Lo->sz_oto;
        info->result_bytes = Lo->sz_res;
        info->scratch_bytes = Lo->sz_scr;
        info->paper_running_bytes = paper;
        info->n_doubles_per_config = P.nd_cfg;
        info->updates_per_config = (long)upd_cfg;
        info->updates_per_sweep = (long)upd_sweep;
        info->form = spec ? U1ML_FORM_SPECTRAL : U1ML_FORM_HISTORY;
        info->spectral_bytes = Lo->sz_wf + Lo->sz_gf + Lo->sz_sph + Lo->sz_spo + Lo->sz_facc + Lo->sz_saved +
                               Lo->sz_cpl + Lo->sz_opl;
        info->launches_per_config = (long)body_launches(P);
        info->est_history_ms = P.est_hist_ms;
        info->est_spectral_ms = P.est_spec_ms;
        info->ins_slots = (!P.probes.empty() && !P.spectral) ? P.ins_ks : 0;
    }
    return true;
}

}  // namespace

// A lane: a subset of the problem's ensembles with its own descriptors,
// launch tables, results-ring counter, stream and graphs.  The whole batch
// is one lane (used by every call); a batch of two or more ensembles is also
// split into up to four lanes of about equal volume that run sweeps and
// multilevel configurations on as many streams at once.  A checkerboard
// phase of a few tens of MB lasts a few microseconds, most of it the latency
// of its dependent loads and of the launch itself, so phases of different
// lanes running side by side fill the machine where one alone does not, and
// the heatbath phases (bound by arithmetic) of one lane overlap the
// overrelaxation phases (bound by memory) of another.  Each ensemble's
// arithmetic is the same in every lane arrangement.
struct Lane {
    int n = 0;
    std::vector<int> idx;        // problem indices of the lane's ensembles
    std::vector<EnsDesc> h_ens;  // their descriptors, lane order
    std::vector<int> h_bstart;   // kNumTabs x (n + 1)
    std::vector<UpdBlock> h_bmap[kUpdateClasses];  // per-block update records of each class
    std::vector<MeasBlock> h_mmap;  // work-groups of a measurement
    EnsDesc* d_ens = nullptr;
    int* d_bstart = nullptr;
    UpdBlock* d_bmap = nullptr;
    MeasBlock* d_mmap = nullptr;
    int* d_ring = nullptr;
    double* prodpart = nullptr;
    size_t bmap_stride = 0;
    SlabBlock* d_smap[3] = {};
    std::vector<SlabBlock> h_smap[3];  // work-groups of the sweeps in LDS
    PairBlock* d_pmap[kPairClasses] = {};
    std::vector<PairBlock> h_pmap[kPairClasses];  // work-groups of the both-parities launches
    int upd_grid[kUpdateClasses] = {0, 0, 0, 0};  // grid size of each update class (multiple of 8)
    bool span[kUpdateClasses] = {};               // the class's records are SpanBlocks
    int max_s_in = 1;                              // largest number of inner slabs in the lane
    hipStream_t stream = nullptr;
    hipGraphExec_t g_sweep = nullptr, g_ml = nullptr;

    int tab_total(int tab) const { return h_bstart[(size_t)tab * (n + 1) + n]; }
    const int* tab_dev(int tab) const { return d_bstart + (size_t)tab * (n + 1); }
    const UpdBlock* bmap_dev(int cls) const { return d_bmap + (size_t)cls * bmap_stride; }
};

struct u1ml_ctx {
    Problem P;
    Sizes S;
    Layout Lo;
    u1ml_plan_info plan;
    char* ws = nullptr;
    hipStream_t stream = nullptr;
    hipStream_t lane_stream[kMaxLanes] = {};  // streams of lanes 1.. (lane 0 runs on the context's stream)
    hipEvent_t ev_fork = nullptr, ev_join[kMaxLanes] = {};
    int device = 0;
    // device pointers
    void* links = nullptr;
    double2 *hit = nullptr, *hc = nullptr, *at = nullptr, *ato = nullptr, *ot = nullptr, *oto = nullptr;
    void* ho = nullptr;
    double *res = nullptr, *vpart = nullptr, *ppart = nullptr, *pout = nullptr,
           *stage = nullptr;
    ObsDesc* d_obs = nullptr;
    int *d_r = nullptr, *d_probe = nullptr, *d_comp = nullptr;
    int con_block = 64;                            // contraction work-group size
    size_t con_lds = 0;                            // contraction dynamic LDS per work-group
    double2 *wf = nullptr, *gf = nullptr, *sph = nullptr, *spo = nullptr, *facc = nullptr;  // spectral form
    double2* cpl = nullptr;                        // plane-major slab phases of one measurement
    void* opl = nullptr;                           // plane-major O rows of one measurement
    void* saved = nullptr;                         // replay copy of the links
    int spec_npm = 0;                              // largest lattice extent (spectral launches)
    long long spec_n12max = 0;                     // largest transverse plane (sites)
    int spec_tile = 4;                             // plane-transform tile (4, or 2 if an extent is not a multiple of 4)
    int spec_square = -1;                          // side of every plane if all are squares of one side, else 0
    int *d_pgroup = nullptr, *d_gdesc = nullptr, *d_pblk = nullptr;
    PairRow* d_prow = nullptr;  // row tables of the both-parities launches
    size_t ins_lds = 0;  // insertion contraction dynamic LDS per work-group
    int ins_block = 64;  // insertion contraction work-group size
    int ins_line_len = 0;  // sites of every charge-axis line of every ensemble where they are all the same, else 0
    uint32_t* d_upd = nullptr;
    unsigned long long* d_count = nullptr;
    double* static_partials = nullptr;  // the library's static scratch on this context's device
    std::vector<EnsDesc> h_ens;  // descriptors in problem order
    Lane whole;                  // every ensemble
    Lane split[kMaxLanes];       // the lanes (batches of two or more ensembles)
    int n_lanes = 1;             // lanes that sweeps and configurations run on (1: the whole batch)
    int block = 256;
    bool initialised = false;
    int ring_count = 0;
    bool use_graphs = true;
    std::string err;
};

namespace {

// the whole-batch lane and every lane of the split (those not in use have no ensembles)
std::vector<Lane*> all_lanes(u1ml_ctx* c)
{
    std::vector<Lane*> v{&c->whole};
    for (int l = 0; l < kMaxLanes; ++l) v.push_back(&c->split[l]);
    return v;
}

u1ml_status set_err(u1ml_ctx* c, u1ml_status s, const std::string& m)
{
    if (c)
        c->err = m;
    else
        g_err = m;
    return s;
}

#define HIPCHK(ctx, expr)                                                                                    \
    do {                                                                                                     \
        hipError_t _e = (expr);                                                                              \
        if (_e != hipSuccess)                                                                                \
            return set_err((ctx), U1ML_EDEVICE, std::string(#expr) + ": " + hipGetErrorString(_e));          \
    } while (0)

void build_tab(Lane& L, int tab, const std::vector<long long>& items, int block)
{
    int* b = &L.h_bstart[(size_t)tab * (L.n + 1)];
    b[0] = 0;
    for (int e = 0; e < L.n; ++e) b[e + 1] = b[e] + (int)((items[e] + block - 1) / block);
}

void build_update_tabs(const u1ml_ctx* c, Lane& L)
{
    const Problem& P = c->P;
    const int n = L.n;
    // time slices whose links a class updates: temporal, spatial full, spatial inner tau, spatial outer tau
    const int skip[kUpdateClasses] = {0, 0, P.tau_i > 1 ? P.tau_i : 0, P.tau_o > 1 ? P.tau_o : 0};
    std::vector<long long> items(n);
    for (int cls = 0; cls < kUpdateClasses; ++cls) {
        auto slices = [&](const EnsDesc& E) { return (long long)(skip[cls] ? E.nt - E.nt / skip[cls] : E.nt); };
        // Work-groups that span time slices where slices leave more than a tenth of
        // their waves' work-items idle and the launch has more waves than SIMDs (one
        // slice a work-group has shorter addresses: below that, latency counts).  Full
        // sweeps, us, slice by slice / spanning: FP32 4^3 x 16384 367 / 167, 6^3 x 4096
        // 186 / 165, FP64 4^3 x 4096 214 / 175, 2^3 x 131072 6121 / 351.
        long long by_slice = 0, packed = 0;
        for (const EnsDesc& E : L.h_ens) {
            const long long slice = (long long)E.nxh * E.ny * E.nz;
            by_slice += slices(E) * ((slice + 63) / 64);
            packed += (slices(E) * slice + 63) / 64;
        }
        L.span[cls] = by_slice > 4 * 256 && 10 * by_slice > 11 * packed;
        for (int e = 0; e < n; ++e) {
            const EnsDesc& E = L.h_ens[e];
            const long long slice = (long long)E.nxh * E.ny * E.nz;
            items[e] = L.span[cls] ? (slices(E) * slice + c->block - 1) / c->block
                                   : slices(E) * ((slice + c->block - 1) / c->block);
        }
        build_tab(L, kTabUpd + cls, items, 1);
    }
    // Blocks are dealt to the 8 XCDs round-robin (block b runs on XCD b mod 8),
    // and each XCD has its own L2.  Logical block L(b) = (b mod 8) per + b / 8
    // gives every XCD one contiguous stretch of the lattice, so neighbouring
    // rows shared by adjacent blocks are fetched into one L2 instead of
    // several.  Launches have 8 per blocks; entries past the end are idle.
    UpdBlock pad;
    std::memset(&pad, 0, sizeof pad);
    for (auto& m : L.h_bmap) m.clear();
    for (int cls = 0; cls < kUpdateClasses; ++cls) {
        const int total = L.h_bstart[(size_t)(kTabUpd + cls) * (n + 1) + n];
        const int per = (total + kXcds - 1) / kXcds;
        std::vector<UpdBlock> logical;
        logical.reserve(total);
        for (int e = 0; e < n; ++e) {
            const EnsDesc& E = L.h_ens[e];
            if (L.span[cls]) {
                SpanBlock r;
                std::memset(&r, 0, sizeof r);
                r.e = E.res_index;
                r.m = skip[cls] ? skip[cls] - 1 : 0;
                r.nxh = E.nxh;
                r.ny = E.ny;
                r.slice = E.nxh * E.ny * E.nz;
                r.vh = E.vh;
                r.nt = E.nt;
                r.inv_nxh = E.inv_nxh;
                r.inv_ny = E.inv_ny;
                r.inv_slice = E.inv_slice;
                r.link_off = E.link_off;
                const long long links = (long long)r.slice * (r.m ? E.nt - E.nt / skip[cls] : E.nt);
                for (long long k = 0; k < links; k += c->block) {
                    const int u = (int)(k / r.slice);  // the first link's slice among the updated ones
                    r.i0 = (int)(k % r.slice);
                    r.n = (int)std::min<long long>(c->block, links - k);
                    r.r0 = r.m ? u % r.m : 0;
                    r.t0 = r.m ? u / r.m * skip[cls] + 1 + r.r0 : u;
                    UpdBlock b;
                    std::memcpy(&b, &r, sizeof b);
                    logical.push_back(b);
                }
                continue;
            }
            UpdBlock r = pad;
            r.slice = E.nxh * E.ny * E.nz;
            r.nxh = E.nxh;
            r.ny = E.ny;
            r.vh = E.vh;
            r.inv_nxh = E.inv_nxh;
            r.inv_ny = E.inv_ny;
            r.e = E.res_index;
            r.link_off = E.link_off;
            // The order keeps what neighbours share within the XCD's L2 (4 MiB):
            // time slice fastest (the blocks of one stretch of the slice at
            // consecutive times follow each other), then the stretches of a
            // group of rows, then z; the group is sized so that one z step,
            // eight (direction, parity) arrays of it, takes 1 MiB, and only the
            // rows at its ends are fetched twice.  With whole planes per z step
            // (8 MiB) one phase of 128^3 x 16 FP32 fetched 815 MB for 537 MB of
            // distinct words.  Planes that are no whole number of blocks are
            // walked as they lie.
            const int plane = E.nxh * E.ny, word = P.precision == U1ML_FP64 ? 8 : 4;
            const bool grouped = plane % c->block == 0;
            // (a step's bytes reach 2^32 where long time extents meet planes smaller than a work-group)
            const long long bytes = (long long)E.nt * c->block * 8 * word;
            const int step = (int)std::max(1ll, (1 << 20) / bytes) * c->block;
            const int group = grouped ? std::min(step, plane) : r.slice;
            const int nz = grouped ? E.nz : 1, width = grouped ? plane : r.slice;
            for (int g0 = 0; g0 < width; g0 += group)
                for (int z = 0; z < nz; ++z)
                    for (int i = g0; i < std::min(g0 + group, width); i += c->block)
                        for (int t = 0; t < E.nt; ++t) {
                            if (skip[cls] && t % skip[cls] == 0) continue;
                            r.i0 = z * plane + i;
                            const int row = r.i0 / E.nxh;
                            r.x0 = r.i0 % E.nxh;
                            r.y0 = row % E.ny;
                            r.zt = row / E.ny + t;
                            r.t0 = (unsigned)t * (unsigned)r.slice;
                            r.tp = (unsigned)((t + 1) % E.nt) * (unsigned)r.slice;
                            r.tm = (unsigned)((t + E.nt - 1) % E.nt) * (unsigned)r.slice;
                            logical.push_back(r);
                        }
        }
        // padding blocks: a record that starts past its slice (every work-item inactive)
        UpdBlock idle = total > 0 ? logical[total - 1] : pad;
        if (L.span[cls]) {
            SpanBlock none;
            std::memcpy(&none, &idle, sizeof none);
            none.n = 0;
            std::memcpy(&idle, &none, sizeof idle);
        } else {
            idle.i0 = idle.slice;
        }
        for (int phys = 0; phys < per * kXcds; ++phys) {
            const int lg = (phys % kXcds) * per + phys / kXcds;
            L.h_bmap[cls].push_back(lg < total ? logical[lg] : idle);
        }
        L.upd_grid[cls] = per * kXcds;
    }
}

void build_pair_tabs(const u1ml_ctx* c, Lane& L)
{
    const Problem& P = c->P;
    const int word = P.precision == U1ML_FP64 ? 8 : 4;
    for (int cls = 0; cls < kPairClasses; ++cls) {
        L.h_pmap[cls].clear();
        if (!P.pair_on[cls]) continue;
        std::vector<PairBlock> logical;
        for (int e = 0; e < L.n; ++e) {
            const EnsDesc& E = L.h_ens[e];
            const int k = E.res_index;
            const PairGeo G(P.ens[k], cls, P.pair_tau(cls));
            PairBlock r;
            std::memset(&r, 0, sizeof r);
            r.e = k;
            r.nxh = E.nxh;
            r.vh = E.vh;
            r.inv_nxh = E.inv_nxh;
            r.link_off = E.link_off;
            pair_for_tiles(P, cls, k, [&](const int* o, const int* C) {
                r.base = word * E.nxh * (o[0] + E.ny * (o[1] + E.nz * o[2]));
                r.par = o[0] + o[1] + o[2];
                r.row_tab = P.pair_shape.at(G.shape(o, C));
                r.n1 = G.rows(C) * E.nxh;
                r.n2 = C[0] * C[1] * C[2] * E.nxh;
                logical.push_back(r);
            });
        }
        // the XCD-aware order of build_update_tabs; padding blocks have no links
        PairBlock idle = logical.back();
        idle.n1 = idle.n2 = 0;
        const int total = (int)logical.size(), per = (total + kXcds - 1) / kXcds;
        for (int phys = 0; phys < per * kXcds; ++phys) {
            const int lg = (phys % kXcds) * per + phys / kXcds;
            L.h_pmap[cls].push_back(lg < total ? logical[lg] : idle);
        }
    }
}

void build_slab_tabs(const u1ml_ctx* c, Lane& L)
{
    const Problem& P = c->P;
    for (int cls = 0; cls < 3; ++cls) {
        L.h_smap[cls].clear();
        if (!P.slab_on[cls]) continue;
        const int tau = cls == 0 ? 0 : (cls == 1 ? P.tau_i : P.tau_o);
        for (const EnsDesc& E : L.h_ens) {
            SlabBlock r;
            std::memset(&r, 0, sizeof r);
            r.e = E.res_index;
            r.tau = tau;
            r.layers = tau ? tau + 1 : E.nt;
            r.nxh = E.nxh;
            r.ny = E.ny;
            r.slice = E.nxh * E.ny * E.nz;
            r.vh = E.vh;
            r.nt = E.nt;
            r.inv_nxh = E.inv_nxh;
            r.inv_ny = E.inv_ny;
            r.inv_slice = E.inv_slice;
            r.link_off = E.link_off;
            for (r.t0 = 0; r.t0 < E.nt; r.t0 += tau ? tau : E.nt) L.h_smap[cls].push_back(r);
        }
    }
}

// Every launch table of a lane, from its ensembles' descriptors (whose
// contraction and product fields are already set).
void build_lane_tables(const u1ml_ctx* c, Lane& L)
{
    const Problem& P = c->P;
    const int n = L.n;
    L.h_bstart.assign((size_t)kNumTabs * (n + 1), 0);
    build_update_tabs(c, L);
    build_pair_tabs(c, L);
    build_slab_tabs(c, L);
    const size_t R = P.r.size(), NG = P.gdesc.size() / 2;
    std::vector<long long> all(n), meas(n), con(n), comb(n), prod(n), site(n), plane(n), mac(n), stage(n), ins(n);
    L.max_s_in = 1;
    for (int e = 0; e < n; ++e) {
        const EnsDesc& E = L.h_ens[e];
        const int n3[3] = {E.nx, E.ny, E.nz};
        int lines = 0;
        long long n12max = 0;
        for (int i = 0; i < P.n_dirs; ++i) {
            lines = std::max(lines, E.nsig / n3[P.dirs[i]]);
            n12max = std::max<long long>(n12max, E.nsig / n3[P.dirs[i]]);
        }
        const long long npm = std::max(E.nx, std::max(E.ny, E.nz));
        all[e] = 8ll * E.vh;
        meas[e] = (long long)E.nsig * E.s_in;
        con[e] = (lines + E.con_lpb - 1) / E.con_lpb;
        // insertion contraction: (line, slot-block chunk) work-groups of the axis with the most lines
        ins[e] = (!P.probes.empty() && !P.spectral)
                     ? (long long)lines * ((P.pblk.size() / kInsBlkInts + E.ins_pbw - 1) / E.ins_pbw)
                     : 0;
        comb[e] = (long long)P.n_dirs * R * E.s_out * E.nsig;
        prod[e] = (long long)R * prod_groups(P) * E.prod_nch;
        site[e] = (long long)P.n_dirs * R * E.nsig;
        plane[e] = P.spectral ? (long long)P.n_dirs * E.s_in * ((long long)R + 12) * npm : 0;
        mac[e] = P.spectral ? (long long)P.n_dirs * E.s_in * NG * ((n12max + kMacK - 1) / kMacK) : 0;
        // staging: work-groups of kStageTile x kStageTile tiles per (axis, slab), as k_plane_stage decodes them
        stage[e] = P.spectral ? (long long)P.n_dirs * E.s_in * ((E.nx + kStageTile - 1) / kStageTile) *
                                    ((npm + kStageTile - 1) / kStageTile) * npm
                              : 0;
        L.max_s_in = std::max(L.max_s_in, E.s_in);
    }
    build_tab(L, kTabAll, all, 256);
    build_tab(L, kTabMeas, meas, 256);
    build_tab(L, kTabCon, con, 1);
    build_tab(L, kTabComb, comb, 256);
    build_tab(L, kTabProd, prod, 1);
    build_tab(L, kTabSite, site, 256);
    build_tab(L, kTabPlane, plane, 1);
    build_tab(L, kTabMac, mac, 1);
    build_tab(L, kTabStage, stage, 1);
    build_tab(L, kTabIns, ins, 1);
    L.h_mmap.clear();
    const int* b = &L.h_bstart[(size_t)kTabMeas * (n + 1)];
    for (int e = 0; e < n; ++e)
        for (int k = b[e]; k < b[e + 1]; ++k) {
            const EnsDesc& E = L.h_ens[e];
            MeasBlock r;
            std::memset(&r, 0, sizeof r);
            r.e = e;
            r.blk = k - b[e];
            const long long item = 256ll * r.blk;
            r.s0 = (int)(item / E.nsig);
            r.xs0 = (int)(item % E.nsig);
            r.nx = E.nx;
            r.ny = E.ny;
            r.nt = E.nt;
            r.slabs = E.s_in;
            r.nsig = E.nsig;
            r.vh = E.vh;
            r.inv_nx = 0.5f * E.inv_nxh;
            r.inv_ny = E.inv_ny;
            r.inv_nsig = 0.5f * E.inv_slice;
            r.link_off = E.link_off;
            L.h_mmap.push_back(r);
        }
}

hipError_t upload_update_tabs(const Lane& L)
{
    hipError_t e = hipSuccess;
    for (int cls = 0; cls < kUpdateClasses && e == hipSuccess; ++cls)
        if (!L.h_bmap[cls].empty())
            e = hipMemcpy(L.d_bmap + (size_t)cls * L.bmap_stride, L.h_bmap[cls].data(),
                          sizeof(UpdBlock) * L.h_bmap[cls].size(), hipMemcpyHostToDevice);
    return e;
}

hipError_t upload_lane(const Lane& L)
{
    const int ring0[4] = {0, 0, 0, 0};
    hipError_t e = hipMemcpy(L.d_ens, L.h_ens.data(), sizeof(EnsDesc) * L.n, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(L.d_bstart, L.h_bstart.data(), sizeof(int) * L.h_bstart.size(), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = upload_update_tabs(L);
    for (int cls = 0; cls < kPairClasses && e == hipSuccess; ++cls)
        if (!L.h_pmap[cls].empty())
            e = hipMemcpy(L.d_pmap[cls], L.h_pmap[cls].data(), sizeof(PairBlock) * L.h_pmap[cls].size(),
                          hipMemcpyHostToDevice);
    for (int cls = 0; cls < 3 && e == hipSuccess; ++cls)
        if (!L.h_smap[cls].empty())
            e = hipMemcpy(L.d_smap[cls], L.h_smap[cls].data(), sizeof(SlabBlock) * L.h_smap[cls].size(),
                          hipMemcpyHostToDevice);
    if (e == hipSuccess && !L.h_mmap.empty())
        e = hipMemcpy(L.d_mmap, L.h_mmap.data(), sizeof(MeasBlock) * L.h_mmap.size(), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(L.d_ring, ring0, sizeof ring0, hipMemcpyHostToDevice);
    return e;
}

// Splits the batch into nl lanes of about equal volume (largest ensembles
// first, each to the lane with the least volume so far; a lane keeps the
// problem order), builds and uploads their tables.  Lanes past nl, and with
// nl = 1 all of them, are emptied; their device areas stay reserved.  Where it
// fails the context is left with one lane.
hipError_t split_lanes(u1ml_ctx* c, int nl)
{
    c->n_lanes = 1;
    // streams as they are needed: the runtime maps streams to a few hardware
    // queues, and a lane that shares one with the context's stream (or with
    // another context's) waits for it
    for (int l = 1; l < nl; ++l) {
        hipError_t e = hipSuccess;
        if (!c->lane_stream[l]) e = hipStreamCreateWithFlags(&c->lane_stream[l], hipStreamNonBlocking);
        if (e == hipSuccess && !c->ev_join[l]) e = hipEventCreateWithFlags(&c->ev_join[l], hipEventDisableTiming);
        if (e != hipSuccess) return e;
    }
    const int n = c->P.n_ens;
    const Layout& Lo = c->Lo;
    char* s = c->ws + Lo.off_scr;
    std::vector<int> order(n);
    for (int e = 0; e < n; ++e) order[e] = e;
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return c->h_ens[a].vh > c->h_ens[b].vh; });
    std::vector<std::vector<int>> parts(nl);
    std::vector<long long> load(nl, 0);
    for (int e : order) {
        const int l = (int)(std::min_element(load.begin(), load.end()) - load.begin());
        parts[l].push_back(e);
        load[l] += c->h_ens[e].vh;
    }
    size_t pp_off = 0;
    for (int l = 0; l < kMaxLanes; ++l) {
        Lane& L = c->split[l];
        if (L.g_sweep) (void)hipGraphExecDestroy(L.g_sweep);
        if (L.g_ml) (void)hipGraphExecDestroy(L.g_ml);
        L.g_sweep = L.g_ml = nullptr;
        L.idx = nl > 1 && l < nl ? parts[l] : std::vector<int>();  // one lane: the whole-batch lane runs, with its own tables
        std::sort(L.idx.begin(), L.idx.end());
        L.n = (int)L.idx.size();
        L.h_ens.clear();
        for (int e : L.idx) L.h_ens.push_back(c->h_ens[e]);
        L.bmap_stride = Lo.bmap_stride;
        L.d_ens = (EnsDesc*)(s + Lo.s_lens[l]);
        L.d_bstart = (int*)(s + Lo.s_lbstart[l]);
        L.d_bmap = (UpdBlock*)(s + Lo.s_lbmap[l]);
        L.d_mmap = (MeasBlock*)(s + Lo.s_lmmap[l]);
        L.d_ring = (int*)(s + Lo.s_lring[l]);
        for (int cls = 0; cls < kPairClasses; ++cls) L.d_pmap[cls] = (PairBlock*)(s + Lo.s_lpmap[l][cls]);
        for (int cls = 0; cls < 3; ++cls) L.d_smap[cls] = (SlabBlock*)(s + Lo.s_lsmap[l][cls]);
        // the lanes use disjoint parts of the slab-product partials
        L.prodpart = (double*)(s + Lo.s_prodpart) + pp_off;
        L.stream = l == 0 ? c->stream : c->lane_stream[l];
        if (L.n == 0) continue;
        build_lane_tables(c, L);
        pp_off += (size_t)L.tab_total(kTabProd) * kProdQ * 2;
        hipError_t e = upload_lane(L);
        if (e != hipSuccess) return e;
    }
    c->n_lanes = nl;
    return hipSuccess;
}

// Bytes [begin, end) of ensemble k's share of a section whose per-ensemble
// element offsets are off[] (elements of `elem` bytes, `total` bytes in all).
void ens_range(const std::vector<size_t>& off, int k, size_t elem, size_t total, size_t* begin, size_t* end)
{
    *begin = off[k] * elem;
    *end = k + 1 < (int)off.size() ? off[k + 1] * elem : total;
}

// Fill with zeros the shares of the lane's ensembles (a whole-array fill
// would race with the other lane).
hipError_t zero_lane(const Lane& L, void* base, const std::vector<size_t>& off, size_t elem, size_t total,
                     hipStream_t st)
{
    for (int e = 0; e < L.n; ++e) {
        size_t b, en;
        ens_range(off, L.idx[e], elem, total, &b, &en);
        hipError_t r = launch_fill_zero((char*)base + b, en - b, st);
        if (r != hipSuccess) return r;
    }
    return hipSuccess;
}

int update_class(const u1ml_ctx* c, int mu, int tau, bool* ok)
{
    *ok = true;
    if (mu == 3) return 0;
    if (tau <= 1) return 1;
    if (tau == c->P.tau_i) return 2;
    if (tau == c->P.tau_o) return 3;
    *ok = false;
    return -1;
}

// 0: every link updated, 1: inner slabs, 2: outer slabs (tau one of the problem's)
int update_class_tau(const u1ml_ctx* c, int tau) { return tau <= 1 ? 0 : (tau == c->P.tau_i ? 1 : 2); }

constexpr unsigned kInPlace[4] = {0, 0, 0, 0};  // every direction in the first link buffer

hipError_t enq_phase(u1ml_ctx* c, const Lane& L, hipStream_t st, int kind, int mu, int parity, int tau,
                     int pass_offset, const unsigned* src, hipEvent_t ev_start = nullptr,
                     hipEvent_t ev_stop = nullptr)
{
    bool ok;
    const int cls = update_class(c, mu, tau, &ok);
    if (!ok) return hipErrorInvalidValue;
    return launch_update(UpdLaunch{c->whole.d_ens, L.bmap_dev(cls), L.span[cls], L.upd_grid[cls], c->block, c->P.precision, c->links,
                                   c->d_upd, pass_offset, kind, mu, parity, {src[0], src[1], src[2], src[3]},
                                   c->P.metro_delta, st, ev_start, ev_stop});
}

// One pass over the directions, each in both parities.  src: the byte offset
// of each direction's current link buffer; a both-parities launch turns its
// direction's over.
hipError_t enq_pass(u1ml_ctx* c, const Lane& L, hipStream_t st, int kind, int tau, int pass_offset, bool pairs,
                    unsigned* src)
{
    const unsigned alt = (unsigned)c->Lo.off_alt;
    for (int mu = 0; mu < 4; ++mu) {
        const int cls = mu == 3 ? 9 : 3 * mu + update_class_tau(c, tau);
        hipError_t e = hipSuccess;
        if (pairs && c->P.pair_on[cls]) {
            const unsigned dst = src[mu] ? 0u : alt;
            e = launch_pair(PairLaunch{c->whole.d_ens, L.d_pmap[cls], c->d_prow, (int)L.h_pmap[cls].size(),
                                       c->P.pair_block[cls], c->P.precision, c->links, c->d_upd, pass_offset, kind, mu,
                                       {src[0], src[1], src[2], src[3]}, dst, c->P.metro_delta, st});
            src[mu] = dst;
        } else {
            for (int p = 0; p < 2 && e == hipSuccess; ++p)
                e = enq_phase(c, L, st, kind, mu, p, tau, pass_offset, src);
        }
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// one sweep: stochastic pass (heatbath or Metropolis) with counter offset hb,
// then n_or overrelaxation passes.  It starts and ends in the first link
// buffer: of an odd number of passes the last one updates in place.
hipError_t enq_sweep(u1ml_ctx* c, const Lane& L, hipStream_t st, int tau, int hb)
{
    const int stoch = c->P.update == U1ML_UPDATE_METROPOLIS ? U1ML_METROPOLIS : U1ML_HEATBATH;
    const int paired = (c->P.n_or + 1) / 2 * 2;  // passes that may turn the buffers over
    unsigned src[4] = {0, 0, 0, 0};
    hipError_t e = hipSuccess;
    for (int k = 0; e == hipSuccess && k <= c->P.n_or; ++k)
        e = enq_pass(c, L, st, k == 0 ? stoch : U1ML_OVERRELAX, tau, hb, k < paired, src);
    return e;
}

// Before sweeps inside slabs of thickness tau: both link buffers hold the
// frozen links, which are spatial ones.
hipError_t enq_mirror(u1ml_ctx* c, const Lane& L, hipStream_t st, int tau)
{
    bool any = false;
    for (int mu = 0; mu < 3; ++mu) any = any || c->P.pair_on[3 * mu + update_class_tau(c, tau)];
    if (!any) return hipSuccess;
    return launch_mirror(L.d_ens, L.n, c->P.precision, c->links, (unsigned)c->Lo.off_alt, 256, st);
}

// n sweeps, in LDS where the plan has them so (at most kSlabSweeps a launch),
// with counter offsets hb, hb + 1, ...
hipError_t enq_sweeps(u1ml_ctx* c, const Lane& L, hipStream_t st, int tau, int hb, int n)
{
    const Problem& P = c->P;
    const int cls = update_class_tau(c, tau);
    hipError_t e = hipSuccess;
    if (!P.slab_on[cls]) {
        for (int k = 0; e == hipSuccess && k < n; ++k) e = enq_sweep(c, L, st, tau, hb + k);
        return e;
    }
    const int stoch = P.update == U1ML_UPDATE_METROPOLIS ? U1ML_METROPOLIS : U1ML_HEATBATH;
    for (int k = 0; e == hipSuccess && k < n; k += kSlabSweeps)
        e = launch_slab(SlabLaunch{c->whole.d_ens, L.d_smap[cls], (int)L.h_smap[cls].size(), P.slab_block[cls], P.precision,
                                   P.slab_lds_bytes[cls], c->links, c->d_upd, hb + k, std::min(kSlabSweeps, n - k), stoch,
                                   P.n_or, P.metro_delta, st});
    return e;
}

// The n_o outer iterations of Algorithm 1 (one iteration for one level).
//   store_o:  measurements keep the slab sums of O
//   ins_hist: history form: per-site insertion averages, combined per level
//   spec_acc: spectral form: after each inner level, weights G_k and the
//             plane transforms of every stored measurement into the sums
// *hb returns the number of heatbath counter offsets used.
hipError_t enq_levels(u1ml_ctx* c, const Lane& L, hipStream_t st, bool store_o, bool ins_hist, bool spec_acc,
                      int* hb_out)
{
    const Problem& P = c->P;
    const int n = L.n;
    hipError_t e = hipSuccess;
    if (P.two && !spec_acc) {
        e = zero_lane(L, c->ot, c->S.ot, 16, c->Lo.sz_ot, st);
        if (e == hipSuccess && ins_hist) e = zero_lane(L, c->oto, c->S.oto, 16, c->Lo.sz_oto, st);
    }
    int hb = 0;
    for (int ko = 0; e == hipSuccess && ko < P.n_o; ++ko) {
        if (P.two && P.k_o > 0) {
            e = enq_mirror(c, L, st, P.tau_o);
            if (e == hipSuccess) e = enq_sweeps(c, L, st, P.tau_o, hb, P.k_o);
            hb += P.k_o;
        }
        if (e == hipSuccess && P.k_i > 0) e = enq_mirror(c, L, st, P.tau_i);
        for (int m = 0; e == hipSuccess && m < P.n_i; ++m) {
            if (e == hipSuccess) e = enq_sweeps(c, L, st, P.tau_i, hb, P.k_i);
            hb += P.k_i;
            if (e == hipSuccess)
                e = launch_measure(L.d_ens, L.d_mmap, L.tab_total(kTabMeas), P.precision, c->links, c->hit, c->hc, c->ho,
                                   c->vpart, m, ko * P.n_i + m, P.tau_i, store_o ? 1 : 0, P.multihit ? 1 : 0, st);
        }
        if (e == hipSuccess)
            e = launch_contract(L.d_ens, L.tab_dev(kTabCon), n, L.tab_total(kTabCon), c->con_block, c->con_lds,
                                c->d_obs, c->d_r, c->hc, c->at, P.n_i, L.max_s_in, P.n_dirs, st);
        if (e == hipSuccess && ins_hist)
            e = launch_contract_ins(L.d_ens, L.tab_dev(kTabIns), n, L.tab_total(kTabIns), c->ins_block, c->ins_lds,
                                    c->d_obs, c->d_r, c->d_comp, c->d_pblk, P.ins_ks, c->hc, c->ho, c->ato, P.n_i,
                                    P.precision, L.max_s_in, P.n_dirs, c->ins_line_len, st);
        if (e == hipSuccess && P.two && !spec_acc)
            e = launch_combine(L.d_ens, L.tab_dev(kTabComb), n, L.tab_total(kTabComb), c->d_obs, c->at,
                               ins_hist ? c->ato : nullptr, c->ot, ins_hist ? c->oto : nullptr, P.tau_o / P.tau_i, st);
        if (spec_acc) {
            // one level: the weights are relative to 2^E(r) of this level's correlator products
            if (e == hipSuccess && !P.two)
                e = launch_prod_exp(L.d_ens, L.tab_dev(kTabProd), n, L.tab_total(kTabProd), c->d_obs,
                                    (int)P.r.size(), prod_groups(P), c->at, 0, 1.0, L.prodpart, c->res, L.d_ring, st);
            if (e == hipSuccess)
                e = launch_gfac(L.d_ens, L.tab_dev(kTabSite), n, L.tab_total(kTabSite), c->d_obs, c->at,
                                P.two ? c->wf : nullptr, P.two ? P.tau_o / P.tau_i : 0, c->gf, c->res, L.d_ring, st);
            for (int m = 0; e == hipSuccess && m < P.n_i; ++m) {
                e = launch_plane_stage(L.d_ens, L.tab_dev(kTabStage), n, L.tab_total(kTabStage), c->d_obs, c->hc,
                                       c->ho, m, P.precision, c->cpl, c->opl, st);
                if (e == hipSuccess)
                    e = launch_dft_planes(L.d_ens, L.tab_dev(kTabPlane), n, L.tab_total(kTabPlane), c->spec_square,
                                          c->spec_n12max, c->spec_npm, c->d_obs, c->d_r, c->cpl, c->opl, c->gf, c->sph,
                                          c->spo, P.precision, c->spec_tile, st);
                if (e == hipSuccess)
                    e = launch_spec_mac(L.d_ens, L.tab_dev(kTabMac), n, L.tab_total(kTabMac), c->spec_npm,
                                        (int)P.comps.size(), c->d_obs, c->d_r, c->d_comp, c->d_gdesc, c->sph, c->spo,
                                        c->facc, st);
            }
        }
    }
    *hb_out = hb;
    return e;
}

// copies the links of the lane's ensembles (replay of two-level spectral configurations)
hipError_t copy_lane_links(u1ml_ctx* c, const Lane& L, const void* src, void* dst, hipStream_t st)
{
    const size_t word = c->P.precision == U1ML_FP64 ? 8 : 4;
    for (int e = 0; e < L.n; ++e) {
        size_t b, en;
        ens_range(c->S.links, L.idx[e], word, c->Lo.sz_links, &b, &en);
        hipError_t r = launch_copy((const char*)src + b, (char*)dst + b, en - b, st);
        if (r != hipSuccess) return r;
    }
    return hipSuccess;
}

// Body of Algorithm 1 for one configuration of the lane's ensembles.
//  history form: one pass; per-site averages of every probe, then products.
//  spectral form, one level: one pass; after the level the weights
//    W_s = prod_{s' != s} [T] are known and the stored measurements are
//    transformed into the spectral sums.
//  spectral form, two levels: pass 1 computes the correlator, the vacuum
//    sums and the outer averages A (no insertions); the links are restored
//    to the configuration's start and pass 2 repeats the same updates with
//    the same counters (so the same trajectory, bit for bit), forming the
//    spectral sums with G_k = W_S prod [T]_k after every inner level.
hipError_t enq_multilevel(u1ml_ctx* c, const Lane& L, hipStream_t st)
{
    const Problem& P = c->P;
    const int n = L.n;
    const bool probes = !P.probes.empty();
    const int npg = prod_groups(P);
    const int R = (int)P.r.size();
    hipError_t e = hipSuccess;
    int hb = 0;
    auto product = [&](bool ins) {  // ins only in the history form, where npg = number of probes
        if (P.two)
            return launch_product(L.d_ens, L.tab_dev(kTabProd), n, L.tab_total(kTabProd), c->d_obs, R, npg, c->ot,
                                  ins ? c->oto : nullptr, 1, 1.0 / P.n_o, L.prodpart, c->res, L.d_ring, st);
        return launch_product(L.d_ens, L.tab_dev(kTabProd), n, L.tab_total(kTabProd), c->d_obs, R, npg, c->at,
                              ins ? c->ato : nullptr, 0, 1.0, L.prodpart, c->res, L.d_ring, st);
    };
    const long long n_sums = P.probes.empty() ? 0 : (long long)R * P.comps.size() * 2 * (P.gdesc.size() / 2);
    if (!P.spectral) {
        e = enq_levels(c, L, st, probes, probes, false, &hb);
        if (e == hipSuccess) e = product(probes);
        if (e == hipSuccess) e = launch_vac_final(L.d_ens, n, c->d_obs, c->vpart, P.n_o * P.n_i, c->res, L.d_ring, st);
    } else if (!P.two) {
        e = zero_lane(L, c->facc, c->S.facc, 16, c->Lo.sz_facc, st);
        if (e == hipSuccess) e = enq_levels(c, L, st, true, false, true, &hb);
        if (e == hipSuccess) e = product(false);
        if (e == hipSuccess)
            e = launch_spec_final(L.d_ens, n, c->d_obs, n_sums, c->spec_npm, c->spec_n12max, c->d_probe,
                                  c->d_pgroup, c->facc, (double)P.n_i, c->res, L.d_ring, st);
        if (e == hipSuccess) e = launch_vac_final(L.d_ens, n, c->d_obs, c->vpart, P.n_i, c->res, L.d_ring, st);
    } else {
        e = copy_lane_links(c, L, c->links, c->saved, st);
        if (e == hipSuccess) e = enq_levels(c, L, st, false, false, false, &hb);
        if (e == hipSuccess) e = product(false);
        if (e == hipSuccess) e = launch_vac_final(L.d_ens, n, c->d_obs, c->vpart, P.n_o * P.n_i, c->res, L.d_ring, st);
        if (e == hipSuccess)
            e = launch_wfac(L.d_ens, L.tab_dev(kTabSite), n, L.tab_total(kTabSite), c->d_obs, c->ot, 1.0 / P.n_o,
                            c->wf, c->res, L.d_ring, st);
        if (e == hipSuccess) e = copy_lane_links(c, L, c->saved, c->links, st);
        if (e == hipSuccess) e = zero_lane(L, c->facc, c->S.facc, 16, c->Lo.sz_facc, st);
        int hb2 = 0;
        if (e == hipSuccess) e = enq_levels(c, L, st, true, false, true, &hb2);
        if (e == hipSuccess)
            e = launch_spec_final(L.d_ens, n, c->d_obs, n_sums, c->spec_npm, c->spec_n12max, c->d_probe,
                                  c->d_pgroup, c->facc, (double)P.n_o * P.n_i, c->res, L.d_ring, st);
    }
    if (e == hipSuccess) e = launch_ring_advance(L.d_ring, st);
    if (e == hipSuccess && hb > 0) e = launch_advance_counters(L.d_ens, c->d_upd, n, hb, st);
    return e;
}

hipError_t enq_sweep_with_counter(u1ml_ctx* c, const Lane& L, hipStream_t st)
{
    hipError_t e = enq_sweep(c, L, st, 0, 0);
    if (e == hipSuccess) e = launch_advance_counters(L.d_ens, c->d_upd, L.n, 1, st);
    return e;
}

void drop_graphs(u1ml_ctx* c)
{
    for (Lane* L : all_lanes(c)) {
        if (L->g_sweep) (void)hipGraphExecDestroy(L->g_sweep);
        if (L->g_ml) (void)hipGraphExecDestroy(L->g_ml);
        L->g_sweep = L->g_ml = nullptr;
    }
}

// graphs, streams and events of a context, then the context
void release(u1ml_ctx* c)
{
    drop_graphs(c);
    if (c->ev_fork) (void)hipEventDestroy(c->ev_fork);
    for (int l = 0; l < kMaxLanes; ++l) {
        if (c->ev_join[l]) (void)hipEventDestroy(c->ev_join[l]);
        if (c->lane_stream[l]) (void)hipStreamDestroy(c->lane_stream[l]);
    }
    delete c;
}

// Runs body(lane) for the lanes in use, all at once: the streams of lanes
// 1.. wait for the context's stream (lane 0's), and the context's stream
// waits for each of them at the end.  One lane: the whole batch on the
// context's stream.
template <typename F>
hipError_t on_lanes(u1ml_ctx* c, F&& body)
{
    if (c->n_lanes <= 1) return body(c->whole);
    hipError_t e = hipEventRecord(c->ev_fork, c->stream);
    for (int l = 1; l < c->n_lanes && e == hipSuccess; ++l) e = hipStreamWaitEvent(c->lane_stream[l], c->ev_fork, 0);
    for (int l = 0; l < c->n_lanes && e == hipSuccess; ++l) e = body(c->split[l]);
    // the joins are enqueued whatever happened, so no lane stream is left behind
    for (int l = 1; l < c->n_lanes; ++l) {
        hipError_t j = hipEventRecord(c->ev_join[l], c->lane_stream[l]);
        if (j == hipSuccess) j = hipStreamWaitEvent(c->stream, c->ev_join[l], 0);
        if (e == hipSuccess) e = j;
    }
    return e;
}

template <typename F>
u1ml_status capture(u1ml_ctx* c, F&& body, hipGraphExec_t* out)
{
    hipGraph_t g = nullptr;
    const hipStream_t cap = c->lane_stream[1];
    HIPCHK(c, hipStreamBeginCapture(cap, hipStreamCaptureModeRelaxed));
    hipError_t e = body(cap);
    hipError_t e2 = hipStreamEndCapture(cap, &g);
    if (e != hipSuccess) {
        if (g) (void)hipGraphDestroy(g);
        return set_err(c, U1ML_EDEVICE, std::string("kernel launch during capture: ") + hipGetErrorString(e));
    }
    if (e2 != hipSuccess) return set_err(c, U1ML_EDEVICE, std::string("hipStreamEndCapture: ") + hipGetErrorString(e2));
    hipError_t e3 = hipGraphInstantiate(out, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (e3 != hipSuccess) return set_err(c, U1ML_EDEVICE, std::string("hipGraphInstantiate: ") + hipGetErrorString(e3));
    return U1ML_OK;
}

// Streaming-model byte count of one phase: distinct words read + words written.
void phase_words(const u1ml_ensemble& E, int kind, int mu, int parity, int tau, long long* words, long long* updates)
{
    const int n[4] = {E.ns[0], E.ns[1], E.ns[2], E.nt};
    const long long V = (long long)n[0] * n[1] * n[2] * n[3];
    std::vector<unsigned char> rd((size_t)(4 * V), 0);
    long long w = 0, u = 0;
    auto sid = [&](int c[4]) { return (long long)c[0] + n[0] * ((long long)c[1] + n[1] * ((long long)c[2] + (long long)n[2] * c[3])); };
    for (int t = 0; t < n[3]; ++t)
        for (int z = 0; z < n[2]; ++z)
            for (int y = 0; y < n[1]; ++y)
                for (int x = 0; x < n[0]; ++x) {
                    if (((x + y + z + t) & 1) != parity) continue;
                    if (mu < 3 && tau > 1 && t % tau == 0) continue;
                    ++u;
                    int c[4] = {x, y, z, t};
                    if (kind != 0) rd[(size_t)(mu + 4 * sid(c))] = 1;
                    for (int nu = 0; nu < 4; ++nu) {
                        if (nu == mu) continue;
                        int a[4], b[4], d[4], f[4];
                        std::memcpy(a, c, sizeof a);
                        a[mu] = (a[mu] + 1) % n[mu];  // x + mu
                        std::memcpy(b, c, sizeof b);
                        b[nu] = (b[nu] + 1) % n[nu];  // x + nu
                        std::memcpy(d, c, sizeof d);
                        d[nu] = (d[nu] - 1 + n[nu]) % n[nu];  // x - nu
                        std::memcpy(f, a, sizeof f);
                        f[nu] = (f[nu] - 1 + n[nu]) % n[nu];  // x + mu - nu
                        rd[(size_t)(nu + 4 * sid(a))] = 1;
                        rd[(size_t)(mu + 4 * sid(b))] = 1;
                        rd[(size_t)(nu + 4 * sid(c))] = 1;
                        rd[(size_t)(nu + 4 * sid(d))] = 1;
                        rd[(size_t)(nu + 4 * sid(f))] = 1;
                        rd[(size_t)(mu + 4 * sid(d))] = 1;
                    }
                }
    for (unsigned char v : rd) w += v;
    *words = w + u;
    *updates = u;
}

// What an entry point returns for an exception, none of which crosses the
// interface: they come from the containers' allocations.
u1ml_status thrown(u1ml_ctx* c) noexcept
{
    try {
        return set_err(c, U1ML_ENOMEM, "host allocation failed");
    } catch (...) {
        return U1ML_ENOMEM;
    }
}

}  // namespace

// ===========================================================================
// C ABI
// ===========================================================================
extern "C" {

const char* u1ml_status_str(u1ml_status s)
{
    switch (s) {
    case U1ML_OK: return "ok";
    case U1ML_EINVAL: return "invalid argument";
    case U1ML_ENOMEM: return "size overflow or out of host memory";
    case U1ML_EDEVICE: return "HIP device error";
    case U1ML_ESTATE: return "call made in the wrong state";
    case U1ML_ENOTSUP: return "not supported";
    }
    return "unknown status";
}

const char* u1ml_last_error(const u1ml_ctx* ctx) { return ctx ? ctx->err.c_str() : g_err.c_str(); }

u1ml_status u1ml_plan(const u1ml_problem* problem, u1ml_plan_info* out)
try {
    if (!out) return set_err(nullptr, U1ML_EINVAL, "plan output is NULL");
    Problem P;
    std::string err;
    if (!read_problem(problem, &P, &err)) return set_err(nullptr, U1ML_EINVAL, err);
    Sizes S;
    Layout Lo;
    if (!compute_sizes(P, &S, out, &Lo, &err)) return set_err(nullptr, U1ML_ENOMEM, err);
    g_err.clear();
    return U1ML_OK;
} catch (...) {
    return thrown(nullptr);
}

u1ml_status u1ml_create(const u1ml_problem* problem, void* d_ws, size_t ws_bytes, void* hip_stream, u1ml_ctx** out)
try {
    if (!out) return set_err(nullptr, U1ML_EINVAL, "output pointer is NULL");
    *out = nullptr;
    std::unique_ptr<u1ml_ctx, void (*)(u1ml_ctx*)> own(new u1ml_ctx(), release);
    u1ml_ctx* const c = own.get();
    std::string err;
    if (!read_problem(problem, &c->P, &err)) return set_err(nullptr, U1ML_EINVAL, err);
    if (!compute_sizes(c->P, &c->S, &c->plan, &c->Lo, &err)) return set_err(nullptr, U1ML_ENOMEM, err);
    if (!d_ws || ws_bytes < c->plan.ws_bytes)
        return set_err(nullptr, U1ML_EINVAL, "workspace too small: need " + std::to_string(c->plan.ws_bytes) + " bytes");
    if (((uintptr_t)d_ws) % kAlign != 0) return set_err(nullptr, U1ML_EINVAL, "workspace must be 256-byte aligned");
    c->ws = (char*)d_ws;
    c->stream = (hipStream_t)hip_stream;
    hipError_t he = hipGetDevice(&c->device);
    if (he == hipSuccess) he = static_scratch(&c->static_partials);
    // lane 1's stream, also the one that graphs are captured on
    if (he == hipSuccess) he = hipStreamCreateWithFlags(&c->lane_stream[1], hipStreamNonBlocking);
    if (he != hipSuccess) return set_err(nullptr, U1ML_EDEVICE, std::string("stream creation: ") + hipGetErrorString(he));
    const Layout& Lo = c->Lo;
    char* w = c->ws;
    c->links = w + Lo.off_links;
    c->hc = (double2*)(w + Lo.off_hc);
    c->ho = (void*)(w + Lo.off_ho);
    c->at = (double2*)(w + Lo.off_at);
    c->ato = (double2*)(w + Lo.off_ato);
    c->ot = (double2*)(w + Lo.off_ot);
    c->oto = (double2*)(w + Lo.off_oto);
    c->res = (double*)(w + Lo.off_res);
    char* s = w + Lo.off_scr;
    c->d_obs = (ObsDesc*)(s + Lo.s_obs);
    c->d_r = (int*)(s + Lo.s_r);
    c->d_probe = (int*)(s + Lo.s_probe);
    c->d_comp = (int*)(s + Lo.s_comp);
    c->d_upd = (uint32_t*)(s + Lo.s_upd);
    c->vpart = (double*)(s + Lo.s_vpart);
    c->hit = (double2*)(s + Lo.s_hit);
    c->ppart = (double*)(s + Lo.s_ppart);
    c->pout = (double*)(s + Lo.s_pout);
    c->d_count = (unsigned long long*)(s + Lo.s_count);
    c->stage = (double*)(s + Lo.s_stage);
    c->d_pgroup = (int*)(s + Lo.s_pgroup);
    c->d_gdesc = (int*)(s + Lo.s_gdesc);
    c->d_pblk = (int*)(s + Lo.s_pblk);
    c->d_prow = (PairRow*)(s + Lo.s_prow);
    c->wf = (double2*)(w + Lo.off_wf);
    c->gf = (double2*)(w + Lo.off_gf);
    c->sph = (double2*)(w + Lo.off_sph);
    c->spo = (double2*)(w + Lo.off_spo);
    c->facc = (double2*)(w + Lo.off_facc);
    c->cpl = (double2*)(w + Lo.off_cpl);
    c->opl = (void*)(w + Lo.off_opl);
    c->saved = (void*)(w + Lo.off_saved);

    const Problem& P = c->P;
    const int n = P.n_ens;
    c->h_ens.resize(n);
    for (int e = 0; e < n; ++e) {
        const u1ml_ensemble& U = P.ens[e];
        EnsDesc& E = c->h_ens[e];
        std::memset(&E, 0, sizeof E);
        E.nx = U.ns[0];
        E.ny = U.ns[1];
        E.nz = U.ns[2];
        E.nt = U.nt;
        E.nxh = E.nx / 2;
        E.nsig = E.nx * E.ny * E.nz;
        E.vh = E.nsig * E.nt / 2;
        E.s_in = E.nt / P.tau_i;
        E.s_out = P.two ? E.nt / P.tau_o : E.s_in;
        E.n_vac_blocks = (E.nsig * E.s_in + 255) / 256;
        E.inv_nxh = 1.0f / (float)E.nxh;
        E.inv_ny = 1.0f / (float)E.ny;
        E.inv_slice = 1.0f / (float)(E.nxh * E.ny * E.nz);
        E.beta = U.beta;
        E.sqrt_beta = std::sqrt(U.beta);
        E.metro_delta = P.metro_delta;
        E.seed = U.seed;
        E.key_id = U.key_id;
        E.link_off = (long long)c->S.links[e];
        E.hc_off = (long long)c->S.hc[e];
        E.hcm_off = E.hc_off + (long long)P.n_i * E.s_in * E.nsig;
        E.ho_off = (long long)c->S.ho[e];
        E.at_off = (long long)c->S.at[e];
        E.ato_off = (long long)c->S.ato[e];
        E.ot_off = (long long)c->S.ot[e];
        E.oto_off = (long long)c->S.oto[e];
        E.vac_part_off = (long long)c->S.vac[e];
        E.hit_off = (long long)c->S.hit[e];
        E.wf_off = (long long)c->S.wf[e];
        E.gf_off = (long long)c->S.gf[e];
        E.sph_off = (long long)c->S.sph[e];
        E.spo_off = (long long)c->S.spo[e];
        E.facc_off = (long long)c->S.facc[e];
        E.cpl_off = (long long)c->S.cpl[e];
        E.opl_off = (long long)c->S.opl[e];
    }
    ObsDesc O;
    std::memset(&O, 0, sizeof O);
    O.n_dirs = P.n_dirs;
    for (int i = 0; i < 3; ++i) O.dirs[i] = P.dirs[i];
    O.n_r = (int)P.r.size();
    O.n_probe = (int)P.probes.size();
    O.n_comp = (int)P.comps.size();
    O.store_o = P.probes.empty() ? 0 : 1;
    O.n_groups = (int)(P.gdesc.size() / 2);
    O.n_pblocks = (int)(P.pblk.size() / kInsBlkInts);
    O.n_ens_total = n;
    O.multihit = P.multihit ? 1 : 0;
    O.n_doubles_per_config = P.nd_cfg;
    std::vector<int> probe_flat;
    for (const u1ml_probe& p : P.probes) {
        probe_flat.push_back(p.l);
        probe_flat.push_back(p.p1);
        probe_flat.push_back(p.p2);
        probe_flat.push_back(p.mode);
    }
    // Contraction shape: a line of N sites along a charge axis has N * n_r
    // pairs (x, r), one thread each; a work-group of con_block threads holds
    // con_lpb such lines, and stages con_mc measurements at a time in LDS.
    // Insertions: a work-group per (line, slab, axis, ins_pbw slot blocks)
    // with N * ceil(n_r / KR) * ins_pbw tasks, staging ins_mc measurements
    // (the line's phases and the O rows of its slots).
    const size_t R = P.r.size();
    const size_t word = P.precision == U1ML_FP64 ? 8 : 4;  // O history element
    std::vector<int> group(n);
    c->con_block = 256;
    for (int e = 0; e < n; ++e) {
        const EnsDesc& E = c->h_ens[e];
        const int n3[3] = {E.nx, E.ny, E.nz};
        int maxpairs = 0;
        for (int i = 0; i < P.n_dirs; ++i) maxpairs = std::max(maxpairs, n3[P.dirs[i]] * (int)R);
        group[e] = std::min(512, (maxpairs + 63) / 64 * 64);  // the kernel is built for <= 512 threads
        c->con_block = std::max(c->con_block, group[e]);
    }
    c->con_lds = 0;
    for (int e = 0; e < n; ++e) {
        EnsDesc& E = c->h_ens[e];
        const int n3[3] = {E.nx, E.ny, E.nz};
        const size_t nmax = (size_t)std::max(E.nx, std::max(E.ny, E.nz));
        const size_t per = P.multihit ? 32 : 16;  // LDS bytes per (measurement, line site)
        E.con_lpb = c->con_block / group[e];
        const size_t fit = (size_t)kConLds / ((size_t)E.con_lpb * nmax * per);
        E.con_mc = (int)std::max<size_t>(1, std::min<size_t>(fit, (size_t)P.n_i));
        c->con_lds = std::max(c->con_lds, (size_t)E.con_lpb * E.con_mc * nmax * per);
        {
            const int len0 = n3[P.dirs[0]];
            bool same = e == 0 || c->ins_line_len == len0;
            for (int i = 0; i < P.n_dirs; ++i) same = same && n3[P.dirs[i]] == len0;
            c->ins_line_len = same ? len0 : 0;
        }
        if (!P.probes.empty() && !P.spectral && P.ins_ks == kMfSlots) {
            // matrix-core kernel: kMfThreads work-items, (slot block, y, 8
            // separations) tiles, up to 4 kMfTiles per pass over the
            // measurements; as many slot blocks per work-group as one pass
            // holds, fewer while a chunk would hold fewer than 8 measurements;
            // chunks of a multiple of 4 measurements
            const int nsb = (int)(P.pblk.size() / kInsBlkInts);
            const int unit = (int)(nmax * ((R + 7) / 8));
            const int cap = (kMfThreads / 64) * kMfTiles;
            E.ins_pbw = std::max(1, std::min(std::min(nsb, cap / std::max(1, unit)), kMfRows / (2 * kMfSlots)));
            auto fit_mc = [&](int bpw) {
                int mc = (std::min(P.n_i, kMfPh) + 3) / 4 * 4;
                while (mc > 4 && !mf_chunk_fits(mc, (int)nmax, (int)R, bpw * 2 * kMfSlots, (int)word)) mc -= 4;
                return mc;
            };
            while (E.ins_pbw > 1 && (!mf_chunk_fits(4, (int)nmax, (int)R, E.ins_pbw * 2 * kMfSlots, (int)word) ||
                                     fit_mc(E.ins_pbw) < std::min(8, (P.n_i + 3) / 4 * 4)))
                --E.ins_pbw;
            const int mc = fit_mc(E.ins_pbw);
            if (!mf_chunk_fits(mc, (int)nmax, (int)R, E.ins_pbw * 2 * kMfSlots, (int)word))
                return set_err(nullptr, U1ML_ENOTSUP, "history-form insertions: matrix-core chunk does not fit LDS");
            c->ins_block = kMfThreads;
            E.ins_mc = mc;
        } else if (!P.probes.empty() && !P.spectral) {
            const int nsb = (int)(P.pblk.size() / kInsBlkInts);
            const int kr = ins_kr(P.ins_ks);
            const int unit = (int)(nmax * ((R + kr - 1) / kr));  // tasks of one slot block
            if (!ins_shape(P, P.ins_ks, nsb, (int)nmax, &E.ins_pbw, &E.ins_mc))
                return set_err(nullptr, U1ML_ENOTSUP,
                               "history-form insertions: one measurement of a work-group's phases or O rows exceeds "
                               "its LDS buffer (use the spectral form)");
            c->ins_block = std::max(c->ins_block, std::min(kInsThreads, (E.ins_pbw * unit + 63) / 64 * 64));
        }
        E.prod_nch = (P.n_dirs * E.nsig + kProdChunk - 1) / kProdChunk;
        E.res_index = e;
        long long n12max = 0;
        for (int i = 0; i < P.n_dirs; ++i) n12max = std::max<long long>(n12max, E.nsig / n3[P.dirs[i]]);
        c->spec_npm = std::max(c->spec_npm, std::max(E.nx, std::max(E.ny, E.nz)));
        c->spec_n12max = std::max(c->spec_n12max, n12max);
        for (int i = 0; i < P.n_dirs; ++i)
            for (int k = 1; k < 3; ++k)
                if (n3[(P.dirs[i] + k) % 3] % 4 != 0) c->spec_tile = 2;
        for (int i = 0; i < P.n_dirs; ++i)
            for (int k = 1; k < 3; ++k) {
                const int n = n3[(P.dirs[i] + k) % 3];
                if (c->spec_square < 0) c->spec_square = n;
                if (c->spec_square != n) c->spec_square = 0;
            }
    }
    // the whole batch as one lane; the split into lanes follows the streams below
    {
        Lane& L = c->whole;
        L.idx.resize(n);
        for (int e = 0; e < n; ++e) L.idx[e] = e;
        L.n = n;
        L.h_ens = c->h_ens;
        L.bmap_stride = Lo.bmap_stride;
        L.d_ens = (EnsDesc*)(s + Lo.s_ens);
        L.d_bstart = (int*)(s + Lo.s_bstart);
        L.d_bmap = (UpdBlock*)(s + Lo.s_bmap);
        L.d_mmap = (MeasBlock*)(s + Lo.s_mmap);
        L.d_ring = (int*)(s + Lo.s_ring);
        for (int cls = 0; cls < kPairClasses; ++cls) L.d_pmap[cls] = (PairBlock*)(s + Lo.s_pmap[cls]);
        for (int cls = 0; cls < 3; ++cls) L.d_smap[cls] = (SlabBlock*)(s + Lo.s_smap[cls]);
        L.prodpart = (double*)(s + Lo.s_prodpart);
        L.stream = c->stream;
        build_lane_tables(c, L);
    }
    {
        // every dynamic LDS request must fit the device's limit per work-group
        int lds_max = 0;
        hipError_t ea = hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, c->device);
        const size_t dft_lds = P.spectral ? plane_lds(c->spec_n12max, c->spec_npm) : 0;
        const size_t mac_lds = P.spectral ? 2 * spec_mac_lds(c->spec_npm) : 0;  // both kinds: the form's limit on the extents
        const size_t slab_bytes = *std::max_element(P.slab_lds_bytes, P.slab_lds_bytes + 3);
        const size_t need = std::max({c->con_lds, c->ins_lds, dft_lds, mac_lds, slab_bytes});
        if (ea != hipSuccess || (size_t)lds_max < need)
            return set_err(nullptr, ea != hipSuccess ? U1ML_EDEVICE : U1ML_ENOTSUP,
                           "work-group LDS of " + std::to_string(need) + " bytes exceeds the device limit of " +
                               std::to_string(lds_max));
    }
    std::vector<uint32_t> zeros(n, 0u);
    u1ml_status st = U1ML_OK;
    auto up = [&](void* dst, const void* src, size_t bytes) {
        if (st != U1ML_OK || bytes == 0) return;
        hipError_t e = hipMemcpy(dst, src, bytes, hipMemcpyHostToDevice);
        if (e != hipSuccess) st = set_err(nullptr, U1ML_EDEVICE, std::string("upload: ") + hipGetErrorString(e));
    };
    up(c->d_obs, &O, sizeof O);
    up(c->d_r, P.r.data(), sizeof(int) * P.r.size());
    up(c->d_probe, probe_flat.data(), sizeof(int) * probe_flat.size());
    up(c->d_comp, P.comps.data(), sizeof(int) * P.comps.size());
    up(c->d_pgroup, P.pgroup.data(), sizeof(int) * P.pgroup.size());
    up(c->d_gdesc, P.gdesc.data(), sizeof(int) * P.gdesc.size());
    up(c->d_pblk, P.pblk.data(), sizeof(int) * P.pblk.size());
    const std::vector<PairRow> prow = build_pair_rows(P);
    up(c->d_prow, prow.data(), sizeof(PairRow) * prow.size());
    up(c->d_upd, zeros.data(), sizeof(uint32_t) * n);
    if (st == U1ML_OK) {
        hipError_t e = upload_lane(c->whole);
        if (e != hipSuccess) st = set_err(nullptr, U1ML_EDEVICE, std::string("upload: ") + hipGetErrorString(e));
    }
    if (st == U1ML_OK) {
        hipError_t e = hipEventCreateWithFlags(&c->ev_fork, hipEventDisableTiming);
        if (e == hipSuccess) e = split_lanes(c, default_lanes(P.ens, P.precision));
        if (e != hipSuccess) st = set_err(nullptr, U1ML_EDEVICE, std::string("lanes: ") + hipGetErrorString(e));
    }
    if (st != U1ML_OK) return st;
    *out = own.release();
    return U1ML_OK;
} catch (...) {
    return thrown(nullptr);
}

u1ml_status u1ml_destroy(u1ml_ctx* ctx)
try {
    if (!ctx) return U1ML_OK;
    // every lane joins the context's stream, so this waits for all work that
    // still reads the workspace or runs the graphs about to be destroyed
    const hipError_t e = hipStreamSynchronize(ctx->stream);
    release(ctx);
    return e == hipSuccess ? U1ML_OK : set_err(nullptr, U1ML_EDEVICE, std::string("u1ml_destroy: ") + hipGetErrorString(e));
} catch (...) {
    return thrown(nullptr);  // (the context is gone)
}

u1ml_status u1ml_init_links(u1ml_ctx* ctx, int start)
try {
    if (!ctx) return set_err(nullptr, U1ML_EINVAL, "ctx is NULL");
    if (start != U1ML_COLD && start != U1ML_HOT) return set_err(ctx, U1ML_EINVAL, "start must be 0 (cold) or 1 (hot)");
    HIPCHK(ctx, launch_init_links(ctx->whole.d_ens, ctx->whole.tab_dev(kTabAll), ctx->P.n_ens, ctx->whole.tab_total(kTabAll),
                                  ctx->P.precision, ctx->links, start, ctx->stream));
    HIPCHK(ctx, launch_fill_zero(ctx->d_upd, align_up(sizeof(uint32_t) * ctx->P.n_ens), ctx->stream));
    ctx->initialised = true;
    return U1ML_OK;
} catch (...) {
    return thrown(ctx);
}

u1ml_status u1ml_sweeps(u1ml_ctx* ctx, int n)
try {
    if (!ctx) return set_err(nullptr, U1ML_EINVAL, "ctx is NULL");
    if (n < 0) return set_err(ctx, U1ML_EINVAL, "n must be >= 0");
    if (!ctx->initialised) return set_err(ctx, U1ML_ESTATE, "links not initialised");
    if (n == 0) return U1ML_OK;
    // one lane's n sweeps on its stream (graph of one sweep, launched n times)
    auto lane_sweeps = [&](Lane& L) -> hipError_t {
        if (ctx->P.slab_on[0]) {  // one launch for many sweeps
            const hipError_t e = enq_sweeps(ctx, L, L.stream, 0, 0, n);
            return e == hipSuccess ? launch_advance_counters(L.d_ens, ctx->d_upd, L.n, n, L.stream) : e;
        }
        if (ctx->use_graphs) {
            if (!L.g_sweep &&
                capture(ctx, [&](hipStream_t st) { return enq_sweep_with_counter(ctx, L, st); }, &L.g_sweep) != U1ML_OK)
                return hipErrorUnknown;
            for (int i = 0; i < n; ++i) {
                hipError_t e = hipGraphLaunch(L.g_sweep, L.stream);
                if (e != hipSuccess) return e;
            }
            return hipSuccess;
        }
        for (int i = 0; i < n; ++i) {
            hipError_t e = enq_sweep_with_counter(ctx, L, L.stream);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    };
    const std::string before = ctx->err;
    hipError_t e = on_lanes(ctx, lane_sweeps);
    if (e != hipSuccess)
        return ctx->err != before && e == hipErrorUnknown ? U1ML_EDEVICE
                                                          : set_err(ctx, U1ML_EDEVICE, std::string("sweeps: ") + hipGetErrorString(e));
    return U1ML_OK;
} catch (...) {
    return thrown(ctx);
}

u1ml_status u1ml_phase(u1ml_ctx* ctx, int kind, int mu, int parity, int tau, int pass_offset)
try {
    if (!ctx) return set_err(nullptr, U1ML_EINVAL, "ctx is NULL");
    if (!ctx->initialised) return set_err(ctx, U1ML_ESTATE, "links not initialised");
    if ((kind < 0 || kind > 2) || mu < 0 || mu > 3 || (parity != 0 && parity != 1) || pass_offset < 0)
        return set_err(ctx, U1ML_EINVAL, "bad phase arguments");
    bool ok;
    update_class(ctx, mu, tau, &ok);
    if (!ok) return set_err(ctx, U1ML_EINVAL, "tau must be <= 1 or one of the problem's level thicknesses");
    HIPCHK(ctx, enq_phase(ctx, ctx->whole, ctx->stream, kind, mu, parity, tau, pass_offset, kInPlace));
    return U1ML_OK;
} catch (...) {
    return thrown(ctx);
}

u1ml_status u1ml_multilevel(u1ml_ctx* ctx)
try {
    if (!ctx) return set_err(nullptr, U1ML_EINVAL, "ctx is NULL");
    if (!ctx->initialised) return set_err(ctx, U1ML_ESTATE, "links not initialised");
    if (ctx->ring_count >= ctx->P.max_configs)
        return set_err(ctx, U1ML_ESTATE, "results ring is full: call u1ml_copy_results");
    const bool graph = ctx->use_graphs && body_phases(ctx->P) <= kMaxGraphPhases;
    auto lane_config = [&](Lane& L) -> hipError_t {
        if (!graph) return enq_multilevel(ctx, L, L.stream);
        if (!L.g_ml && capture(ctx, [&](hipStream_t st) { return enq_multilevel(ctx, L, st); }, &L.g_ml) != U1ML_OK)
            return hipErrorUnknown;
        return hipGraphLaunch(L.g_ml, L.stream);
    };
    const std::string before = ctx->err;
    hipError_t e = on_lanes(ctx, lane_config);
    if (e != hipSuccess)
        return ctx->err != before && e == hipErrorUnknown
                   ? U1ML_EDEVICE
                   : set_err(ctx, U1ML_EDEVICE, std::string("multilevel: ") + hipGetErrorString(e));
    ctx->ring_count++;
    return U1ML_OK;
} catch (...) {
    return thrown(ctx);
}

u1ml_status u1ml_copy_results(u1ml_ctx* ctx, double* host, size_t n_doubles, size_t* n_written)
try {
    if (!ctx) return set_err(nullptr, U1ML_EINVAL, "ctx is NULL");
    if (!host && n_doubles) return set_err(ctx, U1ML_EINVAL, "host is NULL");
    HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
    const size_t avail = (size_t)ctx->ring_count * ctx->P.n_ens * (size_t)ctx->P.nd_cfg;
    const size_t nw = std::min(avail, n_doubles);
    if (nw) HIPCHK(ctx, hipMemcpy(host, ctx->res, nw * sizeof(double), hipMemcpyDeviceToHost));
    int zero[4] = {0, 0, 0, 0};
    for (Lane* L : all_lanes(ctx))
        if (L->n) HIPCHK(ctx, hipMemcpy(L->d_ring, zero, sizeof zero, hipMemcpyHostToDevice));
    ctx->ring_count = 0;
    if (n_written) *n_written = nw;
    return U1ML_OK;
} catch (...) {
    return thrown(ctx);
}

u1ml_status u1ml_get_links(u1ml_ctx* ctx, int ens, double* host, size_t n)
try {
    if (!ctx) return set_err(nullptr, U1ML_EINVAL, "ctx is NULL");
    if (ens < 0 || ens >= ctx->P.n_ens) return set_err(ctx, U1ML_EINVAL, "ensemble index out of range");
    const long long V = 2ll * ctx->h_ens[ens].vh;
    if (!host || n != (size_t)(4 * V)) return set_err(ctx, U1ML_EINVAL, "host buffer must hold exactly 4 V doubles");
    HIPCHK(ctx, launch_gather_links(ctx->whole.d_ens, ens, ctx->P.precision, ctx->links, ctx->stage, V, ctx->stream));
    HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
    HIPCHK(ctx, hipMemcpy(host, ctx->stage, sizeof(double) * 4 * V, hipMemcpyDeviceToHost));
    return U1ML_OK;
} catch (...) {
    return thrown(ctx);
}

u1ml_status u1ml_set_links(u1ml_ctx* ctx, int ens, const double* host, size_t n)
try {
    if (!ctx) return set_err(nullptr, U1ML_EINVAL, "ctx is NULL");
    if (ens < 0 || ens >= ctx->P.n_ens) return set_err(ctx, U1ML_EINVAL, "ensemble index out of range");
    const long long V = 2ll * ctx->h_ens[ens].vh;
    if (!host || n != (size_t)(4 * V)) return set_err(ctx, U1ML_EINVAL, "host buffer must hold exactly 4 V doubles");
    HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
    HIPCHK(ctx, hipMemcpy(ctx->stage, host, sizeof(double) * 4 * V, hipMemcpyHostToDevice));
    HIPCHK(ctx, launch_scatter_links(ctx->whole.d_ens, ens, ctx->P.precision, ctx->links, ctx->stage, V, ctx->stream));
    HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
    ctx->initialised = true;
    return U1ML_OK;
} catch (...) {
    return thrown(ctx);
}

u1ml_status u1ml_get_counter(u1ml_ctx* ctx, int ens, uint32_t* counter)
try {
    if (!ctx) return set_err(nullptr, U1ML_EINVAL, "ctx is NULL");
    if (ens < 0 || ens >= ctx->P.n_ens || !counter) return set_err(ctx, U1ML_EINVAL, "bad arguments");
    HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
    HIPCHK(ctx, hipMemcpy(counter, ctx->d_upd + ens, sizeof(uint32_t), hipMemcpyDeviceToHost));
    return U1ML_OK;
} catch (...) {
    return thrown(ctx);
}

u1ml_status u1ml_set_counter(u1ml_ctx* ctx, int ens, uint32_t counter)
try {
    if (!ctx) return set_err(nullptr, U1ML_EINVAL, "ctx is NULL");
    if (ens < 0 || ens >= ctx->P.n_ens) return set_err(ctx, U1ML_EINVAL, "bad arguments");
    HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
    HIPCHK(ctx, hipMemcpy(ctx->d_upd + ens, &counter, sizeof(uint32_t), hipMemcpyHostToDevice));
    return U1ML_OK;
} catch (...) {
    return thrown(ctx);
}

u1ml_status u1ml_plaquette(u1ml_ctx* ctx, double* out)
try {
    if (!ctx) return set_err(nullptr, U1ML_EINVAL, "ctx is NULL");
    if (!out) return set_err(ctx, U1ML_EINVAL, "out is NULL");
    if (!ctx->initialised) return set_err(ctx, U1ML_ESTATE, "links not initialised");
    HIPCHK(ctx, launch_plaquette(ctx->whole.d_ens, ctx->P.n_ens, 0, ctx->P.precision, ctx->links, ctx->ppart, ctx->pout,
                                 ctx->stream));
    HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
    HIPCHK(ctx, hipMemcpy(out, ctx->pout, sizeof(double) * 6 * ctx->P.n_ens, hipMemcpyDeviceToHost));
    return U1ML_OK;
} catch (...) {
    return thrown(ctx);
}

u1ml_status u1ml_plaquette_noalloc(u1ml_ctx* ctx, double* d_out)
try {
    if (!ctx) return set_err(nullptr, U1ML_EINVAL, "ctx is NULL");
    if (!d_out) return set_err(ctx, U1ML_EINVAL, "d_out is NULL");
    if (ctx->P.n_ens > kStaticPlaqEns)
        return set_err(ctx, U1ML_EINVAL,
                       "u1ml_plaquette_noalloc takes at most " + std::to_string(kStaticPlaqEns) + " ensembles");
    if (!ctx->initialised) return set_err(ctx, U1ML_ESTATE, "links not initialised");
    HIPCHK(ctx, launch_plaquette(ctx->whole.d_ens, ctx->P.n_ens, 0, ctx->P.precision, ctx->links,
                                 ctx->static_partials, d_out, ctx->stream));
    return U1ML_OK;
} catch (...) {
    return thrown(ctx);
}

u1ml_status u1ml_health(u1ml_ctx* ctx, uint64_t* n_bad)
try {
    if (!ctx) return set_err(nullptr, U1ML_EINVAL, "ctx is NULL");
    if (!n_bad) return set_err(ctx, U1ML_EINVAL, "n_bad is NULL");
    HIPCHK(ctx, launch_fill_zero(ctx->d_count, 16, ctx->stream));
    HIPCHK(ctx, launch_health(ctx->whole.d_ens, ctx->whole.tab_dev(kTabAll), ctx->P.n_ens, ctx->whole.tab_total(kTabAll),
                              ctx->P.precision, ctx->links, ctx->d_count, ctx->stream));
    HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
    unsigned long long v = 0;
    HIPCHK(ctx, hipMemcpy(&v, ctx->d_count, sizeof v, hipMemcpyDeviceToHost));
    *n_bad = v;
    return U1ML_OK;
} catch (...) {
    return thrown(ctx);
}

u1ml_status u1ml_set_block(u1ml_ctx* ctx, int block)
try {
    if (!ctx) return set_err(nullptr, U1ML_EINVAL, "ctx is NULL");
    if (block != 64 && block != 128 && block != 256 && block != 512 && block != 1024)
        return set_err(ctx, U1ML_EINVAL, "block must be 64, 128, 256, 512 or 1024");
    HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
    // every lane's tables before the first is replaced: a failed call changes nothing
    std::vector<Lane*> lanes = all_lanes(ctx);
    std::vector<Lane> built;
    const int old = std::exchange(ctx->block, block);
    try {
        for (Lane* L : lanes) {
            built.push_back(*L);
            if (L->n) build_update_tabs(ctx, built.back());
        }
    } catch (...) {
        ctx->block = old;
        throw;
    }
    for (size_t l = 0; l < lanes.size(); ++l) {
        *lanes[l] = std::move(built[l]);
        const Lane& L = *lanes[l];
        if (!L.n) continue;
        HIPCHK(ctx, hipMemcpy(L.d_bstart, L.h_bstart.data(), sizeof(int) * 4 * (L.n + 1), hipMemcpyHostToDevice));
        HIPCHK(ctx, upload_update_tabs(L));
    }
    drop_graphs(ctx);
    return U1ML_OK;
} catch (...) {
    return thrown(ctx);
}

u1ml_status u1ml_set_lanes(u1ml_ctx* ctx, int n_lanes)
try {
    if (!ctx) return set_err(nullptr, U1ML_EINVAL, "ctx is NULL");
    if (n_lanes < 1 || n_lanes > kMaxLanes) return set_err(ctx, U1ML_EINVAL, "n_lanes must be 1, 2, 3 or 4");
    if (n_lanes > ctx->P.n_ens) return set_err(ctx, U1ML_EINVAL, "more lanes than ensembles");
    HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
    // the lanes then in use continue the results ring where it stands (the
    // whole batch as well: it is in use if the split fails)
    const int ring[4] = {ctx->ring_count, 0, 0, 0};
    HIPCHK(ctx, hipMemcpy(ctx->whole.d_ring, ring, sizeof ring, hipMemcpyHostToDevice));
    if (n_lanes != ctx->n_lanes) HIPCHK(ctx, split_lanes(ctx, n_lanes));
    for (Lane* L : all_lanes(ctx))
        if (L->n) HIPCHK(ctx, hipMemcpy(L->d_ring, ring, sizeof ring, hipMemcpyHostToDevice));
    return U1ML_OK;
} catch (...) {
    return thrown(ctx);
}

u1ml_status u1ml_get_lanes(u1ml_ctx* ctx, int* n_lanes)
try {
    if (!ctx) return set_err(nullptr, U1ML_EINVAL, "ctx is NULL");
    if (!n_lanes) return set_err(ctx, U1ML_EINVAL, "n_lanes is NULL");
    *n_lanes = ctx->n_lanes;
    return U1ML_OK;
} catch (...) {
    return thrown(ctx);
}

u1ml_status u1ml_set_graphs(u1ml_ctx* ctx, int enable)
try {
    if (!ctx) return set_err(nullptr, U1ML_EINVAL, "ctx is NULL");
    ctx->use_graphs = enable != 0;
    return U1ML_OK;
} catch (...) {
    return thrown(ctx);
}

namespace {
// Average device time of n_rep launches of one phase by lane L on the
// context's stream, each launch with its own start/stop event pair.
u1ml_status time_lane_phase(u1ml_ctx* ctx, const Lane& L, int kind, int mu, int parity, int tau, int n_rep, double* us)
{
    if (!us || n_rep < 1 || kind < 0 || kind > 2 || mu < 0 || mu > 3 || (parity & ~1))
        return set_err(ctx, U1ML_EINVAL, "bad arguments");
    if (!ctx->initialised) return set_err(ctx, U1ML_ESTATE, "links not initialised");
    bool ok;
    update_class(ctx, mu, tau, &ok);
    if (!ok) return set_err(ctx, U1ML_EINVAL, "tau must be <= 1 or one of the problem's level thicknesses");
    // every launch carries its own start/stop events, which take the dispatch's
    // begin and end timestamps: the average is the kernel's own duration, the
    // figure a kernel trace reports, without the launch gaps between dispatches
    std::vector<hipEvent_t> ev(2 * (size_t)n_rep, nullptr);
    for (auto& x : ev) HIPCHK(ctx, hipEventCreate(&x));
    hipError_t he = hipSuccess;
    for (int i = 0; i < n_rep && he == hipSuccess; ++i)
        he = enq_phase(ctx, L, ctx->stream, kind, mu, parity, tau, 0, kInPlace, ev[2 * i], ev[2 * i + 1]);
    if (he == hipSuccess) he = hipEventSynchronize(ev.back());
    double total = 0.0;
    for (int i = 0; i < n_rep && he == hipSuccess; ++i) {
        float ms = 0.f;
        he = hipEventElapsedTime(&ms, ev[2 * i], ev[2 * i + 1]);
        total += ms;
    }
    for (auto& x : ev) (void)hipEventDestroy(x);
    if (he != hipSuccess) return set_err(ctx, U1ML_EDEVICE, std::string("time_phase: ") + hipGetErrorString(he));
    *us = 1000.0 * total / n_rep;
    return U1ML_OK;
}
}  // namespace

u1ml_status u1ml_time_phase(u1ml_ctx* ctx, int kind, int mu, int parity, int tau, int n_rep, double* us)
try {
    if (!ctx) return set_err(nullptr, U1ML_EINVAL, "ctx is NULL");
    return time_lane_phase(ctx, ctx->whole, kind, mu, parity, tau, n_rep, us);
} catch (...) {
    return thrown(ctx);
}

u1ml_status u1ml_time_phase_lane(u1ml_ctx* ctx, int lane, int kind, int mu, int parity, int tau, int n_rep,
                                 double* us, double* bytes, long* updates)
try {
    if (!ctx) return set_err(nullptr, U1ML_EINVAL, "ctx is NULL");
    if (lane < 0 || lane >= ctx->n_lanes) return set_err(ctx, U1ML_EINVAL, "lane out of range");
    if (!bytes || !updates) return set_err(ctx, U1ML_EINVAL, "bad arguments");
    const Lane& L = ctx->n_lanes <= 1 ? ctx->whole : ctx->split[lane];
    const u1ml_status st = time_lane_phase(ctx, L, kind, mu, parity, tau, n_rep, us);
    if (st != U1ML_OK) return st;
    const double word = ctx->P.precision == U1ML_FP64 ? 8.0 : 4.0;
    double b = 0;
    long u = 0;
    for (int e : L.idx) {
        long long w, uu;
        phase_words(ctx->P.ens[e], kind, mu, parity, tau, &w, &uu);
        b += w * word;
        u += (long)uu;
    }
    *bytes = b;
    *updates = u;
    return U1ML_OK;
} catch (...) {
    return thrown(ctx);
}

u1ml_status u1ml_phase_bytes(u1ml_ctx* ctx, int kind, int mu, int parity, int tau, double* bytes, long* updates)
try {
    if (!ctx) return set_err(nullptr, U1ML_EINVAL, "ctx is NULL");
    if (!bytes || !updates || mu < 0 || mu > 3 || (parity & ~1) || kind < 0 || kind > 2)
        return set_err(ctx, U1ML_EINVAL, "bad arguments");
    const double word = ctx->P.precision == U1ML_FP64 ? 8.0 : 4.0;
    double b = 0;
    long u = 0;
    for (const u1ml_ensemble& E : ctx->P.ens) {
        long long w, uu;
        phase_words(E, kind, mu, parity, tau, &w, &uu);
        b += w * word;
        u += (long)uu;
    }
    *bytes = b;
    *updates = u;
    return U1ML_OK;
} catch (...) {
    return thrown(ctx);
}

u1ml_status u1ml_autotune(u1ml_ctx* ctx, u1ml_tune_report* report)
try {
    if (!ctx) return set_err(nullptr, U1ML_EINVAL, "ctx is NULL");
    if (!ctx->initialised) return set_err(ctx, U1ML_ESTATE, "links not initialised");
    const int cand[5] = {64, 128, 256, 512, 1024};
    HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
    // save links and counters so tuning leaves no trace
    const size_t lbytes = ctx->Lo.sz_links;
    std::vector<uint32_t> upd(ctx->P.n_ens);
    void* saved = nullptr;
    HIPCHK(ctx, hipMalloc(&saved, lbytes));
    hipError_t he = hipMemcpy(saved, ctx->links, lbytes, hipMemcpyDeviceToDevice);
    if (he == hipSuccess) he = hipMemcpy(upd.data(), ctx->d_upd, sizeof(uint32_t) * upd.size(), hipMemcpyDeviceToHost);
    if (he != hipSuccess) {
        (void)hipFree(saved);
        return set_err(ctx, U1ML_EDEVICE, std::string("autotune save: ") + hipGetErrorString(he));
    }
    const int old_block = ctx->block;
    const bool old_graphs = ctx->use_graphs;
    ctx->use_graphs = false;
    double best = 1e300;
    int best_b = old_block;
    u1ml_tune_report rep;
    std::memset(&rep, 0, sizeof rep);
    u1ml_status st = U1ML_OK;
    const int tau = ctx->P.tau_i;
    for (int i = 0; i < 5 && st == U1ML_OK; ++i) {
        st = u1ml_set_block(ctx, cand[i]);
        if (st != U1ML_OK) break;
        hipEvent_t a, b;
        if (hipEventCreate(&a) != hipSuccess || hipEventCreate(&b) != hipSuccess) {
            st = set_err(ctx, U1ML_EDEVICE, "event creation failed");
            break;
        }
        hipError_t e = enq_mirror(ctx, ctx->whole, ctx->stream, tau);
        if (e == hipSuccess) e = enq_sweeps(ctx, ctx->whole, ctx->stream, tau, 0, 1);  // warm-up
        if (e == hipSuccess) e = hipEventRecord(a, ctx->stream);
        for (int k = 0; k < 5 && e == hipSuccess; ++k) e = enq_sweeps(ctx, ctx->whole, ctx->stream, tau, 0, 1);
        if (e == hipSuccess) e = hipEventRecord(b, ctx->stream);
        if (e == hipSuccess) e = hipEventSynchronize(b);
        float ms = 0.f;
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, a, b);
        (void)hipEventDestroy(a);
        (void)hipEventDestroy(b);
        if (e != hipSuccess) {
            st = set_err(ctx, U1ML_EDEVICE, std::string("autotune: ") + hipGetErrorString(e));
            break;
        }
        rep.block[i] = cand[i];
        rep.us_per_sweep[i] = 1000.0 * ms / 5;
        rep.n_candidates = i + 1;
        if (rep.us_per_sweep[i] < best) {
            best = rep.us_per_sweep[i];
            best_b = cand[i];
        }
    }
    hipError_t e1 = hipMemcpy(ctx->links, saved, lbytes, hipMemcpyDeviceToDevice);
    hipError_t e2 = hipMemcpy(ctx->d_upd, upd.data(), sizeof(uint32_t) * upd.size(), hipMemcpyHostToDevice);
    (void)hipFree(saved);
    ctx->use_graphs = old_graphs;
    if (st != U1ML_OK) {
        u1ml_set_block(ctx, old_block);
        return st;
    }
    if (e1 != hipSuccess || e2 != hipSuccess) return set_err(ctx, U1ML_EDEVICE, "autotune restore failed");
    // without a launch of one phase in the sweep the candidates are the same
    bool single = ctx->P.n_or % 2 == 0;  // the last of an odd number of passes
    for (int mu = 0; mu < 4; ++mu) single = single || !ctx->P.pair_on[mu == 3 ? 9 : 3 * mu + 1];
    if (ctx->P.slab_on[1] || !single) best_b = old_block;
    st = u1ml_set_block(ctx, best_b);
    rep.chosen_block = best_b;
    if (report) *report = rep;
    return st;
} catch (...) {
    return thrown(ctx);
}

u1ml_status u1ml_philox_fill(uint32_t k0, uint32_t k1, uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, size_t n,
                             uint32_t* d_out, void* hip_stream)
try {
    if (!d_out && n) return set_err(nullptr, U1ML_EINVAL, "d_out is NULL");
    if (n > 0xFFFFFFFFull) return set_err(nullptr, U1ML_EINVAL, "n must be < 2^32");
    hipError_t e = launch_philox_fill(k0, k1, c0, c1, c2, c3, n, d_out, (hipStream_t)hip_stream);
    if (e != hipSuccess) return set_err(nullptr, U1ML_EDEVICE, hipGetErrorString(e));
    return U1ML_OK;
} catch (...) {
    return thrown(nullptr);
}

u1ml_status u1ml_sincos_fill(const double* d_x, size_t n, double* d_s, double* d_c, void* hip_stream)
try {
    if ((!d_x || !d_s || !d_c) && n) return set_err(nullptr, U1ML_EINVAL, "NULL device pointer");
    if (n > 0xFFFFFFFFull) return set_err(nullptr, U1ML_EINVAL, "n must be < 2^32");
    hipError_t e = launch_sincos_fill(d_x, n, d_s, d_c, (hipStream_t)hip_stream);
    if (e != hipSuccess) return set_err(nullptr, U1ML_EDEVICE, hipGetErrorString(e));
    return U1ML_OK;
} catch (...) {
    return thrown(nullptr);
}

u1ml_status u1ml_vonmises_fill(double kappa, int precision, uint32_t seed, uint32_t key_id, uint32_t c0, uint32_t c1,
                               size_t n, double* d_out, int* d_attempts, void* hip_stream)
try {
    if (!d_out && n) return set_err(nullptr, U1ML_EINVAL, "d_out is NULL");
    if (!(kappa >= 0) || !std::isfinite(kappa)) return set_err(nullptr, U1ML_EINVAL, "kappa must be finite and >= 0");
    if (precision != U1ML_FP64 && precision != U1ML_FP32) return set_err(nullptr, U1ML_EINVAL, "bad precision");
    if (n > 0xFFFFFFFFull) return set_err(nullptr, U1ML_EINVAL, "n must be < 2^32");
    hipError_t e = launch_vonmises_fill(kappa, precision, seed, key_id, c0, c1, n, d_out, d_attempts,
                                        (hipStream_t)hip_stream);
    if (e != hipSuccess) return set_err(nullptr, U1ML_EDEVICE, hipGetErrorString(e));
    return U1ML_OK;
} catch (...) {
    return thrown(nullptr);
}

}  // extern "C"
