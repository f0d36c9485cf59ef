// count.hip -- the host driver of the pair counts (single and batched): work
// list, launch, final merge.  The kernel is in count_kernel.h.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <type_traits>

#include "count_kernel.h"
#include "worklist.h"

namespace fcfc {

// 128-bit fixed-point sums -> FP64, rounded to nearest even, times 2^-S
__global__ void k_finalize_w(const unsigned long long* __restrict__ acc, int nbins, int S, double* __restrict__ out) {
    int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= nbins) return;
    unsigned long long lo = acc[2 * b], hi = acc[2 * b + 1];
    __int128 v = (__int128)(((unsigned __int128)hi << 64) | (unsigned __int128)lo);
    bool neg = v < 0;
    unsigned __int128 m = neg ? (unsigned __int128)(-(v + 1)) + 1u : (unsigned __int128)v;
    double r;
    if (m == 0) {
        r = 0.0;
    } else {
        unsigned long long mh = (unsigned long long)(m >> 64), ml = (unsigned long long)m;
        int nb = mh ? 128 - __clzll(mh) : 64 - __clzll(ml);
        if (nb <= 53) {
            r = ldexp((double)ml, -S);
        } else {
            int sh = nb - 53;
            unsigned __int128 top = m >> sh;
            unsigned __int128 rem = m - (top << sh);
            unsigned __int128 half = (unsigned __int128)1 << (sh - 1);
            if (rem > half || (rem == half && (top & 1u))) top += 1u;
            r = ldexp((double)(unsigned long long)top, sh - S);
        }
    }
    out[b] = neg ? -r : r;
}

static int al16(int b) { return (b + 15) & ~15; }
static size_t al256(size_t b) { return (b + 255) & ~(size_t)255; }

// ---------------------------------------------------------------------------
// host-side preparation shared by the single and batched drivers
// ---------------------------------------------------------------------------
// B points per work item by default, and where the list has to stay short
constexpr int BCHUNK = 2048, BCHUNK_LONG = 16384;

struct LaunchSetup {
    CountArgs a;  // LDS layout and numeric constants (device pointers bound later)
    int waves = 16, T = 128, seg = 1, bchunk = BCHUNK, copies = 1;
    std::vector<int4> rows;
    int nrows = 0;
    std::vector<char> htab;  // tables blob: lut1, lut2, band1, band2, E1, E2, stencil rows
    int lut_entries = 0;     // entries of the look-up table used for s (or s_perp)
    size_t tb_l1 = 0, tb_l2 = 0, tb_b1 = 0, tb_b2 = 0, tb_e1 = 0, tb_e2 = 0, tb_rows = 0, tb_total = 0;
    CountKernel kern = nullptr;
};

// Common fixed-point scale 2^S making every weight product an integer.
static fcfc_status weight_scale(double wmin1, double wmax1, double wmin2, double wmax2, int* S) {
    return weight_scale_rule(wmin1, wmax1, wmin2, wmax2, 2, S);
}

// Most cells a tile may span, unless tuned: 32, so that tiles are cut by
// their point count and fill every lane.  B ranges are trimmed to the tile's
// actual x extent, so a wide tile costs only its extent (measured on MI355X:
// C5 7.0 -> 5.6 ms, C2 8.5 -> 8.3 ms against the earlier density-based span).
static int tile_seg(const Plan* p) { return p->tune.seg_cells > 0 ? std::min(32, p->tune.seg_cells) : 32; }

// The constants of the candidate filter.  It works on points in a frame
// centred on the A points, each coordinate within a few u (2^-24) times the
// extent W of the pair's surroundings, and on |a|^2 - 2 a.b + |b|^2, whose
// terms are below W^2: the error stays below some 70 u W^2, and the margin
// taken is 128 u W^2 (and 64 u W on the second axis).  The coordinates of a
// tree are rounded relative to their leaf's origin, which may lie at a distance
// X far beyond W (a few points along a beam fill one leaf): each component is
// off by another 3 u X at most, the square by 10.4 u X W, and the margins are
// 128 u W (W + X) and 64 u (W + X).  Only pairs truly in range have to pass:
// bin_queue decides.
static void set_filter(const Plan* p, CountArgs& a) {
    const double u = 5.9604644775390625e-08;
    const double up = 1.0 + 1e-6;
    // the reach is 16 to 32 units (as far as a unit's square is a normal FP32 number)
    const int e = std::min(std::max(ilogb(p->rprune) - 4, -62), 59);
    const double sig = ldexp(1.0, -e), sig2 = sig * sig;
    a.f_sig = (float)sig;
    a.f_inv = (float)(1.0 / sig);
    a.f_inv2 = (float)(1.0 / sig2);
    const double e1 = p->e1.back();
    a.f_reach = (float)(p->rprune * up);
    a.f_ext = p->tune.tree_leaf > 0 ? (float)(p->tree_side * up) : 0.f;
    a.f_slack = (float)(128.0 * u);
    a.f_uslack = (float)(64.0 * u);
    double t2 = e1 * e1, cull2 = e1 * e1, ul = 0.0, er = 0.0;
    if (p->kind == FCFC_BIN_SPERP_PI) {
        ul = p->e2.back();
        if (p->los == FCFC_LOS_MIDPOINT) {
            cull2 = p->rprune * p->rprune;
            er = 64.0 * u * sqrt(3.0) * p->coord_max;  // distances from the observer
        }
    }
    a.f_t2 = (float)(t2 * up * sig2);
    a.f_cull2 = (float)(cull2 * up * sig2);
    a.f_u = (float)(ul * up * sig);
    a.f_uerr = (float)(er * up * sig);
    a.f_ts = (float)(4.0 * ul * er * up * sig2);
}

// Uniform edges on every axis: the constants of the computed bins.  The
// separation s32 = Q32 rsq(Q32) of the FP32 displacement is off by at most
//   sqrt(3) e = A / 2   (triangle inequality, e the error of one axis),
//   C s / 2             (rounding of the squares and sums),
//   (TRANS_REL + 2 u) s (rsq, product),
// and the mid-point s_perp, whose square is a difference with an absolute
// error B besides, by B / s32 more (|sqrt x - sqrt y| <= |x - y| / sqrt y).
// x is that over ds, with the rounding of its fma and the distance of the
// edges from e_0 + k ds.  A pair at s32 = 0 gives a NaN and is rechecked.
static void set_linear(const Plan* p, CountArgs& a) {
    const double u = 5.9604644775390625e-08, M = 1.5;
    const bool two = p->kind == FCFC_BIN_SPERP_PI;
    auto uniform = [](const std::vector<double>& e, double* ds, double* off) {
        const int n = (int)e.size() - 1;
        *ds = (e[n] - e[0]) / n;
        *off = 0.0;
        for (int k = 0; k <= n; k++) *off = std::max(*off, fabs(e[k] - (e[0] + k * *ds)));
        return *off <= 1e-9 * *ds;
    };
    double ds1 = 1.0, of1 = 0.0, ds2 = 1.0, of2 = 0.0;
    a.lin = uniform(p->e1, &ds1, &of1) && (!two || uniform(p->e2, &ds2, &of2)) ? 1 : 0;
    if (!a.lin) return;
    const double s1 = p->e1.back() * 1.01, o1 = 1.0 - p->e1[0] / ds1;
    a.e_unit = (float)(u / p->e_axis * (1.0 + 1e-6));
    a.l1c = (float)(1.0 / ds1);
    a.l1o = (float)(o1 - 1.0);
    const double tr = trans_rel_bound();
    const double abs1 = M * (p->em1.A + p->em1.C * s1) / 2.0 + (tr + 4.0 * u) * s1;
    a.l1t = (float)(1.01 * (abs1 + of1) / ds1 + 8.0 * u * (p->n1 + 1.0 + fabs(o1)));
    a.l1a = (float)(1.01 * p->em1.B / ds1);
    a.zero2 = two && p->e2[0] == 0.0;
    if (two) {
        const double o2 = 1.0 - p->e2[0] / ds2, p2 = p->e2.back() * 1.01;
        a.l2c = (float)(1.0 / ds2);
        a.l2o = (float)(o2 - 1.0);
        a.l2t = (float)(1.01 * (M * p->e_pi + M * (tr + 8.0 * u) * p2 + of2) / ds2 + 8.0 * u * (p->n2 + 1.0 + fabs(o2)));
    }
    // bands wider than a quarter of a bin would recheck everything: the tables then
    if (!(a.l1t < 0.25f) || (two && !(a.l2t < 0.25f))) a.lin = 0;
}

// The mu axis: what mu n2 is formed with, and its band around interior edges.
static void set_mu(const Plan* p, bool lin, CountArgs& a) {
    const float shrink = mu_shrink(p->los == FCFC_LOS_MIDPOINT);
    a.mu_n = (float)p->n2;
    a.mu_c = lin ? a.mu_n * (1.0f - shrink) : a.mu_n;
    // one mu bin has no interior edge: nothing is near one
    a.tolA = a.tolC = 0.0f;
    if (p->kind != FCFC_BIN_S_MU || p->n2 < 2) return;
    // pairs closer than sqrt(d2small) are always rechecked: the band then spans a whole mu bin
    a.tolA = std::max(p->mu_tolA, 1.01f * sqrtf(p->d2small));
    a.tolC = p->mu_tolC + (lin ? 1.01f * shrink * a.mu_n : 0.0f);
}

// Format of the weighted words (add_weight) for products p with p 2^S integer
// and |p| <= pmax.  A wave may test `limit` pairs and one more batch (at most
// 79 staged B points x 64, and the rechecks waiting) before the words have to
// be empty again, and 16 waves share them: 16 (limit + 5,248) <= 2^N.  The wider
// the weights, the smaller N and the more often the words go out: on MI355X 1M
// points in 4,000 bins, weights all equal (N = 23) 6,500 times and 4.54 ms, of
// ratio 3 15,900 and 4.62, of ratio 20 (N = 20, about the widest taken) 34,800
// and 4.73 (three words a bin, emptied after 2^26 pairs of a wave: 6.26).
static void set_weight(CountArgs& a, int S, double pmax) {
    int e = 0;
    if (pmax > 0) frexp(pmax, &e);
    const int qb = pmax > 0 ? std::min(62, std::max(53, e + S)) : 53;
    const int N = (124 - qb) / 3;
    WeightFmt& f = a.wf;
    f.k = std::max(qb + N - 62, qb - 50);
    f.cs = f.k + N + 1;
    f.scale = ldexp(1.0, S - f.k);
    f.mul = ldexp(1.0, f.k);
    f.bias = ldexp(1.0, f.k - 1);
    f.one = 1ull << f.cs;
    f.limit = (1u << N) / 16u - 5248u;
}

static fcfc_status setup_launch(Plan* p, bool is_auto, bool weighted, bool batch, LaunchSetup& L) {
    const Grid& g = p->grid;
    const bool tree = p->tune.tree_leaf > 0 && !batch;
    L.T = (tree || p->tune.tile_points != 64) ? 128 : 64;
    L.seg = tile_seg(p);
    // B points per item.  The longest items set the tail of a count whose
    // points crowd into a few cells (row pieces of a few 10^4 points): on
    // MI355X 300k points, 90 % of them in ten blobs, ran 13.0 ms at 16384, 8.3
    // at 4096, 5.9 at 2048, 5.0 at 1024; catalogues without such pieces ran
    // the same at each.  A batch keeps 16384: its list may not outgrow the
    // length sized at creation, and its catalogues fill the chip together.
    L.bchunk = p->tune.b_chunk >= 256 ? p->tune.b_chunk : (batch ? BCHUNK_LONG : BCHUNK);
    L.copies = (p->tune.hist_copies == 2 || p->tune.hist_copies == 4) ? p->tune.hist_copies : 1;
    L.nrows = stencil_rows(p, is_auto, L.rows);
    const bool two = (p->kind == FCFC_BIN_SPERP_PI);
    const bool mid = (p->los == FCFC_LOS_MIDPOINT && p->kind != FCFC_BIN_S);
    const int per_wave = wave_lds_bytes(mid, weighted);
    int dev = 0, maxlds = 65536;
    FCFC_HIP(hipGetDevice(&dev));
    if (hipDeviceGetAttribute(&maxlds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) maxlds = 65536;
    // uniform edges need no look-up table
    CountArgs la;
    memset(&la, 0, sizeof(la));
    set_linear(p, la);
    const bool lin = la.lin != 0;
    const int mode = tree ? COUNT_TREE : batch ? COUNT_BATCH : COUNT_SINGLE;
    L.kern = (lin ? count_kernel_lin : count_kernel_lut)(mode, p->kind, p->los, is_auto, weighted);
    FCFC_HIP(hipFuncSetAttribute((const void*)L.kern, hipFuncAttributeMaxDynamicSharedMemorySize, maxlds));
    // LDS shared by the workgroup's waves for tables of n1t and n2t entries
    auto tables_for = [&](int n1t, int n2t) {
        return al16(n1t * 2 + 4) + al16(n2t * 2 + 4) + al16((p->n1 + 2) * 8) + al16(two ? (p->n2 + 2) * 8 : 0);
    };
    auto shared_for = [&](int n1t, int n2t) {
        return tables_for(n1t, n2t) + (weighted ? al16(p->nbins * 16) : al16(p->nbins * 4 * L.copies));
    };
    // Workgroup size for a given shared part, and the waves resident per CU.
    // Default, from timings on MI355X: two workgroups of 16 or 12 waves per CU
    // when the registers and the LDS allow it, else one workgroup of the
    // largest even wave count that fits (odd counts leave the SIMDs unevenly
    // loaded and ran measurably slower).
    auto choose_waves = [&](int shared, int& waves, int& resident) {
        auto lds_for = [&](int w) { return shared + w * per_wave + 64; };
        if (p->tune.group_waves >= 1 && p->tune.group_waves <= 16) {
            waves = p->tune.group_waves;
            while (waves > 1 && lds_for(waves) > maxlds) waves--;
        } else {
            int two_wg = 0;
            waves = 16;
            while (waves > 1 && lds_for(waves) > maxlds) waves--;
            for (int w : {16, 12}) {
                int occ2 = 0;
                if (lds_for(w) <= maxlds &&
                    hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ2, (const void*)L.kern, w * 64, lds_for(w)) ==
                        hipSuccess &&
                    occ2 >= 2) {
                    two_wg = w;
                    break;
                }
            }
            if (two_wg)
                waves = two_wg;
            else if (waves > 2)
                waves &= ~1;
        }
        int occ = 0;
        if (lds_for(waves) > maxlds ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, (const void*)L.kern, waves * 64, lds_for(waves)) !=
                hipSuccess)
            occ = 0;
        resident = waves * occ;
        return lds_for(waves) <= maxlds;
    };
    // The larger look-up tables (fewer entries that meet a band) are used
    // whenever they keep as many waves resident: on MI355X, when uniform edges
    // read tables too, they ran 20,000 points in s 0.34 -> 0.26 ms and 1M in
    // (s, mu) 5.6 -> 5.3 ms, while costing the weighted count of those two of
    // its 16 waves (7.5 -> 7.8 ms), where they are not used.
    const Lut1D* T1 = &p->lut1;
    const Lut1D* T2 = &p->lut2;
    int shared_bytes = lin ? shared_for(0, 0) : shared_for((int)T1->tab.size(), two ? (int)T2->tab.size() : 0);
    int waves = 1, resident = 0;
    bool fits = choose_waves(shared_bytes, waves, resident);
    // Histograms are accepted up to the size that leaves room for 4 bytes a bin
    // and copy (16 more if weighted), the tables and one wave of MIN_WAVE_LDS,
    // whatever this kernel's waves and bins need: where its larger waves do not
    // fit beside the tables, shorter tables do.
    constexpr int MIN_WAVE_LDS = 3468, MIN_WAVE_LDS_MID = 5248;
    const bool accepted = tables_for((int)T1->tab.size(), two ? (int)T2->tab.size() : 0) +
                              al16(p->nbins * 4 * L.copies) + (weighted ? al16(p->nbins * 16) : 0) +
                              (mid ? MIN_WAVE_LDS_MID : MIN_WAVE_LDS) + 64 <= maxlds;
    Lut1D s1, s2;
    if (accepted && !fits) {
        T1 = &s1;
        T2 = &s2;
        for (int lg = p->tab_log2 - 1; lg >= 0 && !fits; lg--) {
            FCFC_TRY(plan_short_tables(p, lg, s1, s2));
            shared_bytes = shared_for((int)T1->tab.size(), two ? (int)T2->tab.size() : 0);
            fits = choose_waves(shared_bytes, waves, resident);
        }
    } else if (p->has_big && !lin) {
        const int sb = shared_for((int)p->lut1b.tab.size(), two ? (int)p->lut2b.tab.size() : 0);
        int wb = 1, rb = 0;
        if (choose_waves(sb, wb, rb) && rb >= resident && rb > 0) {
            T1 = &p->lut1b;
            T2 = &p->lut2b;
            shared_bytes = sb;
            waves = wb;
        }
    }
    if (!accepted || (!fits && T1 != &p->lut1b)) {
        set_error("count: %d bytes of LDS needed (tables + histogram), device allows %d", shared_bytes + per_wave + 64,
                  maxlds);
        return FCFC_ERANGE;
    }
    L.waves = waves;
    L.lut_entries = lin ? 0 : (int)T1->tab.size();
    CountArgs& a = L.a;
    memset(&a, 0, sizeof(a));
    a.nlut1 = lin ? 0 : (int)T1->tab.size();
    a.nlut2 = two && !lin ? (int)T2->tab.size() : 0;
    a.copies = L.copies;
    int off = 0;
    a.off_lut1 = off;
    off += al16(a.nlut1 * 2 + 4);
    a.off_lut2 = off;
    off += al16(a.nlut2 * 2 + 4);
    a.off_band1 = off;
    off += al16((p->n1 + 2) * 8);
    a.off_band2 = off;
    off += al16(two ? (p->n2 + 2) * 8 : 0);
    a.off_hist = off;
    off += weighted ? 0 : al16(p->nbins * 4 * L.copies);
    a.off_whist = off;
    off += weighted ? al16(p->nbins * 16) : 0;
    a.off_wave = off;
    off += L.waves * per_wave;
    a.off_misc = off;
    off += 64;
    a.lds_bytes = off;
    // tables blob
    L.tb_l1 = (size_t)al16(a.nlut1 * 2 + 4);
    L.tb_l2 = (size_t)al16(a.nlut2 * 2 + 4);
    L.tb_b1 = (size_t)al16((p->n1 + 2) * 8);
    L.tb_b2 = (size_t)al16((p->n2 + 2) * 8);
    L.tb_e1 = (size_t)al16((p->n1 + 1) * 8);
    L.tb_e2 = (size_t)al16((p->n2 + 1) * 8);
    L.tb_rows = (size_t)al16(std::max(1, L.nrows) * 16);
    L.tb_total = L.tb_l1 + L.tb_l2 + L.tb_b1 + L.tb_b2 + L.tb_e1 + L.tb_e2 + L.tb_rows;
    L.htab.assign(L.tb_total, 0);
    {
        size_t o = 0;
        memcpy(&L.htab[o], T1->tab.data(), (size_t)a.nlut1 * 2);
        o += L.tb_l1;
        if (two) memcpy(&L.htab[o], T2->tab.data(), (size_t)a.nlut2 * 2);
        o += L.tb_l2;
        // bands as (lo, hi) pairs, then a sentinel pair above the top edge
        auto put_bands = [&](size_t at, const Lut1D* T, int n) {
            float* b = (float*)&L.htab[at];
            for (int k = 0; k <= n; k++) {
                b[2 * k] = T->lo[k];
                b[2 * k + 1] = T->hi[k];
            }
            b[2 * (n + 1)] = INFINITY;
            b[2 * (n + 1) + 1] = INFINITY;
        };
        put_bands(o, T1, p->n1);
        o += L.tb_b1;
        if (two) put_bands(o, T2, p->n2);
        o += L.tb_b2;
        memcpy(&L.htab[o], T1->E.data(), (p->n1 + 1) * 8);
        o += L.tb_e1;
        if (two) memcpy(&L.htab[o], T2->E.data(), (p->n2 + 1) * 8);
        o += L.tb_e2;
        if (L.nrows) memcpy(&L.htab[o], L.rows.data(), L.nrows * 16);
    }
    // numeric constants
    a.scale1 = T1->scale;
    a.scale2 = two ? T2->scale : 1.f;
    a.vmax1 = T1->vmax;
    a.vmax2 = two ? T2->vmax : 0.f;
    a.n1 = p->n1;
    a.n2 = p->n2;
    a.nbins = p->nbins;
    a.nx = g.nx;
    a.side32 = (float)g.side;
    a.L = g.L;
    a.halfL = g.L * 0.5;
    set_mu(p, lin, a);
    a.mu_top_closed = 1;
    set_filter(p, a);
    set_linear(p, a);
    a.ncat = 1;
    a.flush_pairs = 1ull << (p->tune.flush_log2 >= 1 && p->tune.flush_log2 <= FLUSH_LOG2_MAX ? p->tune.flush_log2
                                                                                              : FLUSH_LOG2_MAX);
    a.shard_count = (p->tune.shard_count >= 1) ? (uint32_t)p->tune.shard_count : 1u;
    a.shard_index = (p->tune.shard_count >= 1) ? (uint32_t)p->tune.shard_index : 0u;
    FCFC_HIP(hipFuncSetAttribute((const void*)L.kern, hipFuncAttributeMaxDynamicSharedMemorySize, a.lds_bytes));
    return FCFC_OK;
}

// Point the table pointers of the arguments into the uploaded blob; returns the stencil rows.
static int4* bind_tables(const LaunchSetup& L, char* tab, CountArgs& a) {
    char* o = tab;
    a.lut1 = (const int16_t*)o;
    o += L.tb_l1;
    a.lut2 = (const int16_t*)o;
    o += L.tb_l2;
    a.band1 = (const float2*)o;
    o += L.tb_b1;
    a.band2 = (const float2*)o;
    o += L.tb_b2;
    a.E1 = (const double*)o;
    o += L.tb_e1;
    a.E2 = (const double*)o;
    o += L.tb_e2;
    return (int4*)o;
}

static WLArgs make_wl(const Plan* p, const LaunchSetup& L, bool is_auto, int ncat, int64_t npoints_a) {
    const Grid& g = p->grid;
    WLArgs w{};
    w.nx = g.nx;
    w.ny = g.ny;
    w.nz = g.nz;
    w.seg = L.seg;
    w.tile = L.T;
    w.bchunk = L.bchunk;
    w.nrows = std::max(1, L.nrows);
    w.periodic = g.L > 0;
    w.is_auto = is_auto;
    w.full_rows = !is_auto;  // stencil_rows keeps the half stencil for auto counts
    w.ncat = ncat;
    // tiles end at `tile` points, at a span of `seg` cells, or at a row end
    const int64_t nrow = (int64_t)g.ny * g.nz * ncat;
    w.tiles_cap = (uint32_t)std::min<int64_t>(nrow * ((g.nx + L.seg - 1) / L.seg + 1) + npoints_a / L.T + 1,
                                              0xffffffffLL);
    return w;
}

// One step of the x order that the sort keys give a row's points.
static float key_xstep(const Grid& g, int xbits) { return (float)(ldexp(g.side, -xbits) * (1.0 + 1e-3)); }

static int grid_blocks(const LaunchSetup& L, uint32_t nitems, int* occ_out = nullptr) {
    int occ = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, (const void*)L.kern, L.waves * 64, L.a.lds_bytes) !=
            hipSuccess ||
        occ < 1)
        occ = 1;
    if (occ_out) *occ_out = occ;
    int64_t nblk = (int64_t)device_cu_count() * occ;
    // a short list is spread over every CU
    int64_t need = std::max<int64_t>(((int64_t)nitems + L.waves - 1) / L.waves,
                                     std::min<int64_t>(nitems, device_cu_count()));
    if (nblk > need) nblk = std::max<int64_t>(1, need);
    return (int)nblk;
}

// sum and maximum over i of 2^pred[i] - 1 (predicted ticks): out[0] += sum;
// out[1] = max, as the bits of a non-negative double (ordered like integers)
__global__ __launch_bounds__(256) void k_sum_exp2m1(const float* __restrict__ pred, uint32_t n, double* out) {
    __shared__ double part[4], pmax[4];
    double acc = 0, mx = 0;
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
        const float v = pred[i];
        const double t = (double)exp2f(fminf(fmaxf(v, 0.f), 40.f)) - 1.0;
        acc += t;
        mx = fmax(mx, t);
    }
    for (int o = 32; o > 0; o >>= 1) {
        acc += __shfl_xor(acc, o);
        mx = fmax(mx, __shfl_xor(mx, o));
    }
    if ((threadIdx.x & 63) == 0) {
        part[threadIdx.x >> 6] = acc;
        pmax[threadIdx.x >> 6] = mx;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        atomicAdd(out, part[0] + part[1] + part[2] + part[3]);
        const double m = fmax(fmax(pmax[0], pmax[1]), fmax(pmax[2], pmax[3]));
        atomicMax((unsigned long long*)(out + 1), (unsigned long long)__double_as_longlong(m));
    }
}

__global__ __launch_bounds__(256) void k_pred_check(const float* __restrict__ pred, uint32_t n,
                                                    unsigned long long* bad) {
    bool b = false;
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) b |= !isfinite(pred[i]);
    if (__any(b) && (threadIdx.x & 63) == 0) atomicOr(bad, 1ull);
}

// k_pred_check over the first *n_dev predictions (a batched list sized on the device)
__global__ __launch_bounds__(256) void k_pred_check_dev(const float* __restrict__ pred, const uint32_t* n_dev,
                                                        unsigned long long* bad) {
    const uint32_t n = *n_dev;
    bool b = false;
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) b |= !isfinite(pred[i]);
    if (__any(b) && (threadIdx.x & 63) == 0) atomicOr(bad, 1ull);
}

// learned sort key: half-octave buckets of the predicted time, longest first;
// the heuristic key (cost = A points x B points) if any prediction was bad
__global__ void k_pred_keys(const Item* __restrict__ items, const float* __restrict__ pred,
                            const unsigned long long* __restrict__ bad, uint32_t n, uint32_t* __restrict__ key,
                            uint32_t* __restrict__ val) {
    uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint32_t k;
    if (*bad) {
        const uint32_t c = items[i].cost;
        const uint32_t lg = c ? 31u - (uint32_t)__clz(c) : 0u;
        const uint32_t half = (lg >= 1 && ((c >> (lg - 1)) & 1u)) ? 1u : 0u;
        k = 63u - min(63u, 2u * lg + half);
    } else {
        const float b = fminf(fmaxf(2.f * pred[i], 0.f), 63.f);
        k = 63u - (uint32_t)b;
    }
    key[i] = k;
    val[i] = i;
}

// ---------------------------------------------------------------------------
// single count
// ---------------------------------------------------------------------------
fcfc_status count_pairs(Plan* p, Cells* c1, Cells* c2, int64_t* d_counts, double* d_wcounts, hipStream_t st,
                        PredictReq* pr, const Workspace* ws) {
    const bool is_auto = (c2 == nullptr);
    Cells* cb = is_auto ? c1 : c2;
    const bool weighted = d_wcounts != nullptr;
    const Grid& g = p->grid;
    const bool tree = c1->tree;
    if (tree != cb->tree || tree != (p->tune.tree_leaf > 0)) {
        set_error("count_pairs: cell sets and plan disagree on grid or tree");
        return FCFC_EGRID;
    }
    if (tree) {
        if (pr) {
            set_error("count_pairs: predictions take grid plans only");
            return FCFC_EINVAL;
        }
        // FP32 bands for leaf-local coordinates: rebuilt when these trees hold
        // points farther from their leaf origins than the bands assume
        const double ext = std::max(c1->tree_ext, cb->tree_ext);
        if (ext > p->tree_side) {
            p->tree_side = ext * (1.0 + 1e-9);
            FCFC_TRY(plan_finalize_numerics(p));
        }
    }
    int S = 0;
    if (weighted) {
        if (!c1->weighted || !cb->weighted) {
            set_error("count_pairs: weighted counts need weights in both cell sets");
            return FCFC_EINVAL;
        }
        FCFC_TRY(weight_scale(c1->wmin, c1->wmax, cb->wmin, cb->wmax, &S));
    }
    LaunchSetup L;
    FCFC_TRY(setup_launch(p, is_auto, weighted, false, L));
    CountArgs& a = L.a;
    if (weighted) set_weight(a, S, c1->wmax * cb->wmax);
    const bool sorted = !pr && p->tune.order != FCFC_ORDER_BUILT;
    const Model* model =
        pr ? pr->model : ((p->tune.order == FCFC_ORDER_LEARNED && !tree) ? p->model : nullptr);
    WLArgs w = make_wl(p, L, is_auto, 1, c1->n);
    w.keyB = cb->xkey;
    w.xbits = cb->xbits;
    // grid: A rows and tiles x stencil rows; tree: A leaves
    const int64_t nseg = tree ? 1 : (int64_t)g.ny * g.nz;
    const int64_t tiles_cap = tree ? 1 : w.tiles_cap;
    if (tiles_cap >= 0xffffffffLL / std::max(1, L.nrows)) {
        set_error("count_pairs: work list too large");
        return FCFC_ERANGE;
    }
    const int64_t npair_tr = tree ? ((int64_t)tree_leaves(c1) << tree_wl_split(c1, cb)) : tiles_cap * w.nrows;

    // scratch 1: tables, tiles, tile counts/offsets, item counts/offsets, counters, arguments
    size_t s_tab = al256(L.tb_total);
    size_t s_tc = al256((size_t)nseg * 4);
    size_t s_tiles = al256((size_t)tiles_cap * sizeof(Tile));
    size_t s_ic = al256((size_t)npair_tr * 4);
    size_t s_scan = al256(std::max(scan_scratch_bytes(nseg), scan_scratch_bytes(npair_tr)));
    size_t s_ctr = 256;
    size_t s_args = al256(sizeof(CountArgs));
    size_t s_acc = weighted ? al256((size_t)p->nbins * 16) : 0;
    size_t s1 = s_tab + 2 * s_tc + s_tiles + 2 * s_ic + s_scan + s_ctr + s_args + s_acc;
    char* scr = nullptr;
    if (ws) {
        // the caller's workspace: nothing is allocated
        if (s1 > ws->bytes) {
            set_error("count_pairs: %zu bytes of scratch needed before the work list, the workspace holds %zu", s1,
                      ws->bytes);
            return FCFC_ERANGE;
        }
        scr = ws->base;
    } else if (dev_alloc((void**)&scr, s1, st) != FCFC_OK) {
        set_error("count_pairs: cannot allocate %zu bytes of scratch", s1);
        return FCFC_ENOMEM;
    }
    auto release = [&](char* ptr) {
        if (!ws) dev_free(ptr, st);
    };
    char* q = scr;
    char* tab = q;
    q += s_tab;
    uint32_t* tcount = (uint32_t*)q;
    q += s_tc;
    uint32_t* toff = (uint32_t*)q;
    q += s_tc;
    Tile* tiles = (Tile*)q;
    q += s_tiles;
    uint32_t* icount = (uint32_t*)q;
    q += s_ic;
    uint32_t* ioff = (uint32_t*)q;
    q += s_ic;
    void* scan_scr = q;
    q += s_scan;
    uint32_t* ctr = (uint32_t*)q;  // [0] ntiles [1] nitems [2] cursor
    q += s_ctr;
    CountArgs* args_dev = (CountArgs*)q;
    q += s_args;
    unsigned long long* wacc = (unsigned long long*)q;

    p->host_stage.swap(L.htab);
    FCFC_HIP(hipMemcpyAsync(tab, p->host_stage.data(), L.tb_total, hipMemcpyHostToDevice, st));
    int4* srows = bind_tables(L, tab, a);
    fill_u32(ctr, 0u, 64, st);
    if (!tree) {
        hipLaunchKernelGGL(k_tile_count, dim3((unsigned)((nseg + 255) / 256)), dim3(256), 0, st, c1->cell_start, w,
                           tcount);
        scan_exclusive_u32(tcount, toff, nseg, &ctr[0], scan_scr, st);
        hipLaunchKernelGGL(k_tile_write, dim3((unsigned)((nseg + 255) / 256)), dim3(256), 0, st, c1->cell_start,
                           c1->xkey, w, toff, tiles);
    }
    // the work list's length, and the scratch it needs
    uint32_t nitems = 0;
    size_t s_items = 0, s_sort = 0, s_rs = 0, s_times = 0, s_pred = 0, s2 = 0;
    for (;;) {
        if (tree)
            tree_items_enqueue(c1, cb, is_auto, p->rprune, p->coord_max, L.bchunk, nullptr, icount, nullptr, 0, st);
        else
            hipLaunchKernelGGL(k_item_count, dim3((unsigned)((npair_tr + 255) / 256)), dim3(256), 0, st, tiles,
                               &ctr[0], srows, cb->cell_start, w, icount);
        scan_exclusive_u32(icount, ioff, npair_tr, &ctr[1], scan_scr, st);
        uint32_t hctr[2] = {0, 0};
        FCFC_HIP(hipMemcpyAsync(hctr, ctr, 8, hipMemcpyDeviceToHost, st));
        FCFC_HIP(hipStreamSynchronize(st));
        nitems = hctr[1];
        s_items = al256((size_t)std::max<uint32_t>(nitems, 1) * sizeof(Item));
        s_sort = sorted ? al256((size_t)std::max<uint32_t>(nitems, 1) * 4) : 0;
        s_rs = sorted ? al256(radix_scratch_bytes(nitems)) : 0;
        s_times = (p->tune.record_timing && !pr && !ws) ? al256((size_t)std::max<uint32_t>(nitems, 1) * 4) : 0;
        s_pred = model ? al256((size_t)std::max<uint32_t>(nitems, 1) * 20) : 0;
        s2 = 2 * s_items + 4 * s_sort + s_rs + s_times + s_pred;
        // a list too long for the caller's workspace is cut into longer items
        if (!ws || s1 + s2 <= ws->bytes || p->tune.b_chunk || L.bchunk == BCHUNK_LONG) break;
        L.bchunk = w.bchunk = BCHUNK_LONG;
    }
    p->last_scratch = s1 + s2;
    char* scr2 = nullptr;
    if (ws) {
        // s1 is a sum of 256-byte multiples, so the second part stays aligned
        if (s1 + s2 > ws->bytes) {
            set_error("count_pairs: %u work items need %zu bytes of scratch, the workspace holds %zu", nitems, s1 + s2,
                      ws->bytes);
            return FCFC_ERANGE;
        }
        scr2 = ws->base + s1;
    } else if (dev_alloc((void**)&scr2, s2, st) != FCFC_OK) {
        dev_free(scr, st);
        set_error("count_pairs: cannot allocate %zu bytes for %u work items", s2, nitems);
        return FCFC_ENOMEM;
    }
    Item* items = (Item*)scr2;
    Item* items2 = (Item*)(scr2 + s_items);
    if (tree)
        tree_items_enqueue(c1, cb, is_auto, p->rprune, p->coord_max, L.bchunk, ioff, nullptr, items, nitems, st);
    else
        hipLaunchKernelGGL(k_item_write, dim3((unsigned)((npair_tr + 255) / 256)), dim3(256), 0, st, tiles, &ctr[0],
                           srows, cb->cell_start, w, ioff, items, nitems);
    Item* run_items = items;
    float* pred = model ? (float*)(scr2 + 2 * s_items + 4 * s_sort + s_rs + s_times) : nullptr;
    const float kcells = (float)(p->rprune / g.side);
    if (pr) {
        // predict-only: score the work list and stop
        const int nblk = grid_blocks(L, nitems);
        double tk[2] = {0, 0};  // predicted ticks: sum, largest item
        if (nitems > 0) {
            model_item_costs(model, items, nitems, kcells, pred + nitems, pred, st);
            double* dsum = (double*)&ctr[8];
            fill_u64((uint64_t*)dsum, 0ull, 2, st);
            hipLaunchKernelGGL(k_sum_exp2m1, dim3(std::min<uint32_t>((nitems + 255) / 256, 1024)), dim3(256), 0, st,
                               pred, nitems, dsum);
            FCFC_HIP(hipMemcpyAsync(tk, dsum, 16, hipMemcpyDeviceToHost, st));
        }
        FCFC_HIP(hipStreamSynchronize(st));
        release(scr2);
        release(scr);
        int khz = 0;
        if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, 0) != hipSuccess || khz <= 0) khz = 100000;
        pr->items = nitems;
        // the schedule can finish no earlier than the mean load of a wave or the largest item
        pr->pred_ms = std::max(tk[0] / ((double)nblk * L.waves), tk[1]) / (double)khz;
        return FCFC_OK;
    }
    // launch statistics: the plan's buffer and events, made by the first
    // allocating count (a count into a workspace keeps none without them)
    if (!p->stats_dev && !ws) {
        FCFC_HIP(hipMalloc(&p->stats_dev, 64));
        FCFC_HIP(hipEventCreate(&p->ev0));
        FCFC_HIP(hipEventCreate(&p->ev1));
    }
    const bool keep_stats = p->stats_dev != nullptr;
    zero_ranges(st, {p->stats_dev, keep_stats ? (size_t)64 : 0}, {d_counts, (size_t)p->nbins * 8},
                {wacc, weighted ? (size_t)p->nbins * 16 : 0});
    if (sorted && nitems > 1) {
        uint32_t* k0 = (uint32_t*)(scr2 + 2 * s_items);
        uint32_t* v0 = (uint32_t*)(scr2 + 2 * s_items + s_sort);
        uint32_t* k1 = (uint32_t*)(scr2 + 2 * s_items + 2 * s_sort);
        uint32_t* v1 = (uint32_t*)(scr2 + 2 * s_items + 3 * s_sort);
        void* rs = scr2 + 2 * s_items + 4 * s_sort;
        if (model) {
            // learned order: longest predicted first; any non-finite prediction
            // sends the whole list back to the heuristic key (flag in stats[5])
            model_item_costs(model, items, nitems, kcells, pred + nitems, pred, st);
            // (ctr[8..9] were zeroed with the other counters)
            unsigned long long* bad = keep_stats ? (unsigned long long*)p->stats_dev + 5 : (unsigned long long*)&ctr[8];
            hipLaunchKernelGGL(k_pred_check, dim3(std::min<uint32_t>((nitems + 255) / 256, 1024)), dim3(256), 0, st,
                               pred, nitems, bad);
            hipLaunchKernelGGL(k_pred_keys, dim3((nitems + 255) / 256), dim3(256), 0, st, items, pred, bad, nitems, k0,
                               v0);
        } else {
            hipLaunchKernelGGL(k_item_keys, dim3((nitems + 255) / 256), dim3(256), 0, st, items, &ctr[1], nitems, k0,
                               v0);
        }
        radix_sort_pairs(&k0, &v0, &k1, &v1, nitems, 8, rs, st);
        hipLaunchKernelGGL(k_item_permute, dim3((nitems + 255) / 256), dim3(256), 0, st, items, v0, &ctr[1], nitems,
                           items2);
        run_items = items2;
    }
    // (none in a caller's workspace: no room is reserved for them there)
    uint32_t* times = s_times ? (uint32_t*)(scr2 + 2 * s_items + 4 * s_sort + s_rs) : nullptr;

    a.posA = c1->pos32;
    a.absA = c1->abs32;
    a.p64A = c1->pos64;
    a.wA = c1->w;
    a.posB = cb->pos32;
    a.p64B = cb->pos64;
    a.wB = cb->w;
    if (tree) {
        a.leaf_orgA = c1->leaf_org;
        a.leaf_orgB = cb->leaf_org;
        a.tree_q = (float)c1->tree_q;
        a.tree_leaf = (uint32_t)cb->xbits;
        a.tree_nleafB = tree_leaves(cb);
    }
    if (!tree) a.xstep = key_xstep(g, c1->xbits);
    a.items = run_items;
    a.nitems_dev = &ctr[1];
    a.cursor = &ctr[2];
    a.out_counts = (unsigned long long*)d_counts;
    a.out_w = weighted ? wacc : nullptr;
    a.stats = keep_stats ? (unsigned long long*)p->stats_dev : nullptr;
    a.times = times;

    int occ = 1;
    const int nblk = grid_blocks(L, nitems, &occ);
    if (keep_stats) FCFC_HIP(hipEventRecord(p->ev0, st));
    p->host_args.resize(sizeof(CountArgs));
    memcpy(p->host_args.data(), &a, sizeof(CountArgs));
    FCFC_HIP(hipMemcpyAsync(args_dev, p->host_args.data(), sizeof(CountArgs), hipMemcpyHostToDevice, st));
    hipLaunchKernelGGL(L.kern, dim3((unsigned)nblk), dim3(L.waves * 64), (size_t)a.lds_bytes, st,
                       (const CountArgs*)args_dev);
    FCFC_HIP(hipGetLastError());
    if (keep_stats) FCFC_HIP(hipEventRecord(p->ev1, st));
    if (weighted)
        hipLaunchKernelGGL(k_finalize_w, dim3((p->nbins + 255) / 256), dim3(256), 0, st, wacc, p->nbins, S, d_wcounts);
    if (times) {
        // keep the per-item times and items for the scheduler (plan-owned)
        if (p->timing_dev) (void)hipFree(p->timing_dev);
        p->timing_dev = nullptr;
        p->timing_n = 0;
        size_t tb = (size_t)nitems * (4 + sizeof(Item));
        if (hipMalloc(&p->timing_dev, std::max<size_t>(tb, 256)) == hipSuccess) {
            FCFC_HIP(hipMemcpyAsync(p->timing_dev, times, (size_t)nitems * 4, hipMemcpyDeviceToDevice, st));
            FCFC_HIP(hipMemcpyAsync((char*)p->timing_dev + (size_t)nitems * 4, run_items, (size_t)nitems * sizeof(Item),
                                    hipMemcpyDeviceToDevice, st));
            p->timing_n = nitems;
        }
    }
    release(scr2);
    release(scr);
    p->last_stream = st;
    p->have_stats = keep_stats;
    p->stats.items = nitems;
    p->stats.cells = tree ? (int64_t)tree_leaves(c1) : g.ncell();
    p->stats.grid[0] = g.nx;
    p->stats.grid[1] = g.ny;
    p->stats.grid[2] = g.nz;
    p->stats.cells_per_rmax = g.k;
    p->stats.cell_side = g.side;
    p->stats.wg_per_cu = occ;
    p->stats.group_waves = L.waves;
    p->stats.lut_entries = L.lut_entries;
    p->stats.order_used = model ? FCFC_ORDER_LEARNED : (sorted ? FCFC_ORDER_HEURISTIC : FCFC_ORDER_BUILT);
    return FCFC_OK;
}

// ---------------------------------------------------------------------------
// batched auto counts of many periodic catalogues
// ---------------------------------------------------------------------------
__global__ void k_clamp_items(uint32_t* ctr, uint32_t cap) {
    if (ctr[1] > cap) {
        ctr[1] = cap;
        ctr[5] = 1u;  // overflow flag
    }
}

struct BatchImpl {
    Plan* plan = nullptr;
    int ncat = 0;
    int npairs = 0;  // histograms written: one per (A, B) catalogue pair
    int xbits = 0;   // sub-cell x bits of the sort keys
    int64_t ntot = 0;
    bool weighted = false;
    int S = 0;
    double wmax = 0;  // largest |weight|
    LaunchSetup L;
    WLArgs wl;
    int64_t nseg = 0, npair_tr = 0;
    uint32_t items_cap = 0;
    int nblk = 1;
    // device
    CatDesc* desc = nullptr;
    int64_t* offs = nullptr;
    uint32_t *key = nullptr, *idx = nullptr, *tk = nullptr, *tv = nullptr;
    uint32_t *key_s = nullptr, *idx_s = nullptr;  // sorted arrays (after ping-pong)
    void* sort_scr = nullptr;
    uint32_t* flags = nullptr;
    uint64_t* wst = nullptr;
    float4* pos32 = nullptr;
    float4* abs32 = nullptr;  // absolute FP32 positions (mid-point line of sight only)
    double* pos64 = nullptr;
    double* w = nullptr;
    uint32_t* cs = nullptr;
    int32_t* pairs = nullptr;  // 2 per pair
    uint32_t *ptile_off = nullptr, *ptile_first = nullptr;
    // largest-first order within each pair: keys, values, sort scratch, sorted items
    uint32_t *sk0 = nullptr, *sv0 = nullptr, *sk1 = nullptr, *sv1 = nullptr;
    // learned order (plan order FCFC_ORDER_LEARNED with a model attached): a
    // frozen copy of the model, item features, predictions, non-finite flag
    Model* msnap = nullptr;
    float* mparams = nullptr;
    float *feat = nullptr, *pred = nullptr;
    unsigned long long* bad = nullptr;
    float kcells = 1.f;
    void* isort_scr = nullptr;
    Item* items2 = nullptr;
    int sort_bits = 8;
    uint32_t key_last = 0;
    uint32_t *tcount = nullptr, *toff = nullptr, *icount = nullptr, *ioff = nullptr;
    void* scan_scr = nullptr;
    Tile* tiles = nullptr;
    Item* items = nullptr;
    uint32_t* ctr = nullptr;  // [0] ntiles [1] nitems [2] cursor [3] nchunks [4] chunk cursor [5] overflow
    unsigned long long* kstats = nullptr;  // counting launch: [0] candidates [1] rechecks [6] early merges
    // pair_items: npairs + 1 item offsets; pair_order: pairs by decreasing estimated cost
    uint32_t *pair_items = nullptr, *pair_order = nullptr, *chunk_prefix = nullptr;
    unsigned long long* counts = nullptr;
    unsigned long long* wacc = nullptr;
    double* wout = nullptr;
    char* tab = nullptr;
    CountArgs* args_dev = nullptr;
    std::vector<void*> allocs;
    std::vector<char> host_args;
    std::vector<uint32_t> host_order;
    std::vector<int32_t> host_pairs;
    std::vector<CatDesc> host_desc;
    std::vector<int64_t> host_offs;
    hipGraph_t graph = nullptr;
    hipGraphExec_t gexec = nullptr;
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    hipStream_t cap = nullptr;  // capture stream (the caller's may be the legacy default stream)
};

static fcfc_status balloc(BatchImpl* b, void** p, size_t bytes) {
    if (hipMalloc(p, std::max<size_t>(bytes, 256)) != hipSuccess) {
        set_error("batch: cannot allocate %zu bytes", bytes);
        return FCFC_ENOMEM;
    }
    b->allocs.push_back(*p);
    return FCFC_OK;
}

void batch_free_impl(BatchImpl* b) {
    if (!b) return;
    model_snapshot_free(b->msnap);
    if (b->gexec) (void)hipGraphExecDestroy(b->gexec);
    if (b->graph) (void)hipGraphDestroy(b->graph);
    if (b->ev0) (void)hipEventDestroy(b->ev0);
    if (b->ev1) (void)hipEventDestroy(b->ev1);
    (void)hipDeviceSynchronize();
    if (b->cap) (void)hipStreamDestroy(b->cap);
    for (void* p : b->allocs) (void)hipFree(p);
    delete b;
}

// Enqueue the build and the work list (up to the item counts).
static void batch_enqueue_front(BatchImpl* b, hipStream_t st) {
    Plan* p = b->plan;
    uint32_t *k = b->key, *v = b->idx, *tk = b->tk, *tv = b->tv;
    batch_build_enqueue(p, b->xbits, b->desc, b->offs, b->ncat, b->ntot, b->weighted, &k, &v, &tk, &tv, b->sort_scr,
                        b->flags, b->wst, b->pos32, b->abs32, b->pos64, b->w, b->cs, st);
    b->key_s = k;
    b->idx_s = v;
    // the sorted keys trim the B ranges (the ping-pong buffer that holds them
    // is the same on every run: the pass count is fixed)
    b->wl.keyB = k;
    b->wl.xbits = b->xbits;
    int4* srows = (int4*)(b->tab + (b->L.tb_total - b->L.tb_rows));
    fill_u32(b->ctr, 0u, 64, st);
    hipLaunchKernelGGL(k_tile_count, dim3((unsigned)((b->nseg + 255) / 256)), dim3(256), 0, st, b->cs, b->wl, b->tcount);
    scan_exclusive_u32(b->tcount, b->toff, b->nseg, &b->ctr[0], b->scan_scr, st);
    hipLaunchKernelGGL(k_tile_write, dim3((unsigned)((b->nseg + 255) / 256)), dim3(256), 0, st, b->cs, k, b->wl,
                       b->toff, b->tiles);
    hipLaunchKernelGGL(k_pair_tiles, dim3(1), dim3(1), 0, st, b->toff, &b->ctr[0], b->wl, b->ptile_off, b->ptile_first);
    hipLaunchKernelGGL(k_item_count, dim3((unsigned)((b->npair_tr + 255) / 256)), dim3(256), 0, st, b->tiles, &b->ctr[0],
                       srows, b->cs, b->wl, b->icount);
    scan_exclusive_u32(b->icount, b->ioff, b->npair_tr, &b->ctr[1], b->scan_scr, st);
}

// Enqueue the rest: items, catalogue ranges, chunks, counting kernel, merge.
static void batch_enqueue_back(BatchImpl* b, hipStream_t st) {
    Plan* p = b->plan;
    int4* srows = (int4*)(b->tab + (b->L.tb_total - b->L.tb_rows));
    hipLaunchKernelGGL(k_clamp_items, dim3(1), dim3(1), 0, st, b->ctr, b->items_cap);
    hipLaunchKernelGGL(k_item_write, dim3((unsigned)((b->npair_tr + 255) / 256)), dim3(256), 0, st, b->tiles, &b->ctr[0],
                       srows, b->cs, b->wl, b->ioff, b->items, b->items_cap);
    hipLaunchKernelGGL(k_pair_items, dim3((b->npairs + 1 + 255) / 256), dim3(256), 0, st, b->ioff, &b->ctr[1], b->wl,
                       b->pair_items);
    // each pair's items largest first (pairs stay in place)
    {
        const unsigned nb = (b->items_cap + 255) / 256;
        uint32_t *k0 = b->sk0, *v0 = b->sv0, *k1 = b->sk1, *v1 = b->sv1;
        if (b->msnap) {
            model_item_costs(b->msnap, b->items, b->items_cap, b->kcells, b->feat, b->pred, st);
            fill_u64((uint64_t*)b->bad, 0ull, 1, st);
            hipLaunchKernelGGL(k_pred_check_dev, dim3(std::min<uint32_t>(nb, 1024)), dim3(256), 0, st, b->pred,
                               &b->ctr[1], b->bad);
            hipLaunchKernelGGL(k_pair_pred_keys, dim3(nb), dim3(256), 0, st, b->items, &b->ctr[1], b->items_cap,
                               b->pair_items, b->npairs, b->key_last, b->pred, b->bad, k0, v0);
        } else {
            hipLaunchKernelGGL(k_pair_item_keys, dim3(nb), dim3(256), 0, st, b->items, &b->ctr[1], b->items_cap,
                               b->pair_items, b->npairs, b->key_last, k0, v0);
        }
        radix_sort_pairs(&k0, &v0, &k1, &v1, b->items_cap, b->sort_bits, b->isort_scr, st);
        hipLaunchKernelGGL(k_item_permute, dim3(nb), dim3(256), 0, st, b->items, v0, &b->ctr[1], b->items_cap,
                           b->items2);
    }
    hipLaunchKernelGGL(k_chunk_prefix, dim3(1), dim3(1), 0, st, b->pair_items, b->pair_order, b->npairs,
                       b->L.a.chunk_items, b->chunk_prefix, &b->ctr[3]);
    zero_ranges(st, {b->counts, (size_t)b->npairs * p->nbins * 8},
                {b->wacc, b->weighted ? (size_t)b->npairs * p->nbins * 16 : 0}, {b->kstats, 64});
    hipLaunchKernelGGL(b->L.kern, dim3((unsigned)b->nblk), dim3(b->L.waves * 64), (size_t)b->L.a.lds_bytes, st,
                       (const CountArgs*)b->args_dev);
    if (b->weighted)
        hipLaunchKernelGGL(k_finalize_w, dim3((b->npairs * p->nbins + 255) / 256), dim3(256), 0, st, b->wacc,
                           b->npairs * p->nbins, b->S, b->wout);
}

fcfc_status batch_create_impl(Plan* p, const fcfc_catalog* cats, int ncat, const int32_t* pairs, int npairs,
                              hipStream_t st, BatchImpl** out) {
    if (p->tune.tree_leaf > 0) {
        set_error("batch_create: batches take grid plans (tree_leaf = 0)");
        return FCFC_EINVAL;
    }
    if (p->L <= 0 && !p->grid_set) {
        set_error("batch_create: an open-box plan needs fcfc_plan_fit_bounds or fcfc_plan_set_bounds first");
        return FCFC_ESTATE;
    }
    BatchImpl* b = new (std::nothrow) BatchImpl();
    if (!b) return FCFC_ENOMEM;
    b->plan = p;
    b->ncat = ncat;
    b->npairs = npairs;
    // weighted when any catalogue has weights; an empty catalogue has no weights to give
    b->weighted = false;
    for (int c = 0; c < ncat; c++) b->weighted = b->weighted || cats[c].w != nullptr;
    b->host_desc.resize(ncat);
    b->host_offs.resize(ncat + 1);
    b->host_pairs.assign(pairs, pairs + 2 * (size_t)npairs);
    int64_t tot = 0;
    for (int c = 0; c < ncat; c++) {
        if (cats[c].n > 0 && (cats[c].w != nullptr) != b->weighted) {
            delete b;
            set_error("batch_create: either every catalogue has weights or none");
            return FCFC_EINVAL;
        }
        b->host_desc[c] = CatDesc{cats[c].xyz, cats[c].w, cats[c].n, tot};
        b->host_offs[c] = tot;
        tot += cats[c].n;
    }
    b->host_offs[ncat] = tot;
    b->ntot = tot;
    if (tot >= ((int64_t)1 << 31)) {
        delete b;
        set_error("batch_create: more than 2^31 points in the batch");
        return FCFC_ERANGE;
    }
    const Grid& g = p->grid;
    if ((int64_t)ncat * g.ncell() >= ((int64_t)1 << 31)) {
        delete b;
        set_error("batch_create: catalogues x cells exceeds 2^31");
        return FCFC_ERANGE;
    }
    bool all_auto = true;
    for (int q = 0; q < npairs; q++) all_auto = all_auto && (pairs[2 * q] == pairs[2 * q + 1]);
    // pair order: largest estimated cost first (n^2 / 2 for an auto count, n_a n_b for a cross count)
    std::vector<double> cost(npairs);
    for (int q = 0; q < npairs; q++) {
        const double na = (double)cats[pairs[2 * q]].n, nb = (double)cats[pairs[2 * q + 1]].n;
        cost[q] = (pairs[2 * q] == pairs[2 * q + 1]) ? 0.5 * na * na : na * nb;
    }
    b->host_order.resize(npairs);
    for (int q = 0; q < npairs; q++) b->host_order[q] = (uint32_t)q;
    std::stable_sort(b->host_order.begin(), b->host_order.end(),
                     [&](uint32_t x, uint32_t y) { return cost[x] > cost[y]; });
    fcfc_status s = setup_launch(p, all_auto, b->weighted, true, b->L);
    if (s != FCFC_OK) {
        delete b;
        return s;
    }
    b->wl = make_wl(p, b->L, all_auto, ncat, tot);
    b->xbits = key_xbits((int64_t)ncat * g.ncell());
    b->nseg = (int64_t)g.ny * g.nz * ncat;  // A rows
    // pair-tiles: every pair takes the tiles of its A catalogue (each bounded as in make_wl)
    std::vector<int64_t> cat_tiles(ncat);
    int64_t tiles = 0;
    for (int c = 0; c < ncat; c++) {
        cat_tiles[c] = (int64_t)g.ny * g.nz * ((g.nx + b->L.seg - 1) / b->L.seg + 1) + cats[c].n / b->L.T + 1;
        tiles += cat_tiles[c];
    }
    int64_t ptiles = 0;
    for (int q = 0; q < npairs; q++) ptiles += cat_tiles[pairs[2 * q]];
    b->npair_tr = ptiles * b->wl.nrows;
    if (tiles >= 0xffffffffLL || b->npair_tr >= 0xffffffffLL) {
        delete b;
        set_error("batch_create: work list too large");
        return FCFC_ERANGE;
    }
    b->wl.npairs = npairs;
    b->wl.ptiles_cap = (uint32_t)ptiles;
    b->wl.tiles_cap = (uint32_t)tiles;
    const int nb = p->nbins;
    const bool need_abs = (p->los == FCFC_LOS_MIDPOINT && p->kind != FCFC_BIN_S);
#define BA(ptr, bytes)                                                         \
    do {                                                                       \
        fcfc_status s_ = balloc(b, (void**)&(ptr), (bytes));                   \
        if (s_ != FCFC_OK) {                                                   \
            batch_free_impl(b);                                                \
            return s_;                                                         \
        }                                                                      \
    } while (0)
    BA(b->desc, sizeof(CatDesc) * ncat);
    BA(b->offs, sizeof(int64_t) * (ncat + 1));
    BA(b->key, 4 * (size_t)tot);
    BA(b->idx, 4 * (size_t)tot);
    BA(b->tk, 4 * (size_t)tot);
    BA(b->tv, 4 * (size_t)tot);
    BA(b->sort_scr, batch_build_scratch(tot));
    BA(b->flags, 64);
    BA(b->wst, STAT_BYTES);
    BA(b->pos32, 16 * (size_t)(tot + 8));
    if (need_abs) BA(b->abs32, 16 * (size_t)(tot + 8));
    BA(b->pos64, 24 * (size_t)tot);
    if (b->weighted) BA(b->w, 8 * (size_t)(tot + 8));
    BA(b->cs, 4 * (size_t)(g.ncell() * ncat + 1));
    BA(b->tcount, 4 * (size_t)b->nseg);
    BA(b->toff, 4 * (size_t)b->nseg);
    BA(b->icount, 4 * (size_t)b->npair_tr);
    BA(b->ioff, 4 * (size_t)b->npair_tr);
    BA(b->scan_scr, std::max(scan_scratch_bytes(b->nseg), scan_scratch_bytes(b->npair_tr)));
    BA(b->tiles, sizeof(Tile) * (size_t)b->wl.tiles_cap);
    BA(b->ctr, 256);
    BA(b->kstats, 64);
    BA(b->pairs, 8 * (size_t)npairs);
    BA(b->ptile_off, 4 * (size_t)(npairs + 1));
    BA(b->ptile_first, 4 * (size_t)npairs);
    BA(b->pair_items, 4 * (size_t)(npairs + 1));
    BA(b->pair_order, 4 * (size_t)npairs);
    BA(b->chunk_prefix, 4 * (size_t)(npairs + 1));
    BA(b->counts, 8 * (size_t)npairs * nb);
    if (b->weighted) {
        BA(b->wacc, 16 * (size_t)npairs * nb);
        BA(b->wout, 8 * (size_t)npairs * nb);
    }
    BA(b->tab, b->L.tb_total);
    BA(b->args_dev, sizeof(CountArgs));
    b->wl.pairs = b->pairs;
    b->wl.ptile_off = b->ptile_off;
    b->wl.ptile_first = b->ptile_first;
    FCFC_HIP(hipMemcpy(b->desc, b->host_desc.data(), sizeof(CatDesc) * ncat, hipMemcpyHostToDevice));
    FCFC_HIP(hipMemcpy(b->offs, b->host_offs.data(), sizeof(int64_t) * (ncat + 1), hipMemcpyHostToDevice));
    FCFC_HIP(hipMemcpy(b->pairs, b->host_pairs.data(), 8 * (size_t)npairs, hipMemcpyHostToDevice));
    FCFC_HIP(hipMemcpy(b->pair_order, b->host_order.data(), 4 * (size_t)npairs, hipMemcpyHostToDevice));
    FCFC_HIP(hipMemcpy(b->tab, b->L.htab.data(), b->L.tb_total, hipMemcpyHostToDevice));
    FCFC_HIP(hipEventCreate(&b->ev0));
    FCFC_HIP(hipEventCreate(&b->ev1));
    // one eager pass of the front half sizes the work list and validates the data
    batch_enqueue_front(b, st);
    uint32_t hctr[2] = {0, 0};
    uint64_t hw[2] = {0, 0};
    std::vector<uint64_t> hws(STAT_SLOTS * STAT_STRIDE);
    uint32_t hflags = 0;
    FCFC_HIP(hipMemcpyAsync(hctr, b->ctr, 8, hipMemcpyDeviceToHost, st));
    FCFC_HIP(hipMemcpyAsync(hws.data(), b->wst, STAT_BYTES, hipMemcpyDeviceToHost, st));
    FCFC_HIP(hipMemcpyAsync(&hflags, b->flags, 4, hipMemcpyDeviceToHost, st));
    FCFC_HIP(hipStreamSynchronize(st));
    if (hflags & 5u) {
        batch_free_impl(b);
        set_error("batch_create: non-finite position or weight");
        return FCFC_ENONFINITE;
    }
    if (hflags & 2u) {
        batch_free_impl(b);
        set_error(p->L > 0 ? "batch_create: a point lies outside [0, L)"
                           : "batch_create: a point lies outside the plan bounds");
        return FCFC_EBOX;
    }
    if (b->weighted) {
        weight_stats_reduce(hws.data(), &hw[0], &hw[1]);
        double wmin = 0, wmax = 0;
        if (hw[0] != ~0ull) memcpy(&wmin, &hw[0], 8);
        memcpy(&wmax, &hw[1], 8);
        b->wmax = wmax;
        fcfc_status ws = weight_scale(wmin, wmax, wmin, wmax, &b->S);
        if (ws != FCFC_OK) {
            batch_free_impl(b);
            return ws;
        }
    }
    b->items_cap = std::max<uint32_t>(hctr[1], 1);
    BA(b->items, sizeof(Item) * (size_t)b->items_cap);
    BA(b->items2, sizeof(Item) * (size_t)b->items_cap);
    BA(b->sk0, 4 * (size_t)b->items_cap);
    BA(b->sv0, 4 * (size_t)b->items_cap);
    BA(b->sk1, 4 * (size_t)b->items_cap);
    BA(b->sv1, 4 * (size_t)b->items_cap);
    BA(b->isort_scr, radix_scratch_bytes(b->items_cap));
    if (p->tune.order == FCFC_ORDER_LEARNED && p->model) {
        BA(b->mparams, model_param_bytes());
        BA(b->feat, 16 * (size_t)b->items_cap);
        BA(b->pred, 4 * (size_t)b->items_cap);
        BA(b->bad, 64);
        b->msnap = model_snapshot(p->model, b->mparams, st);
        if (!b->msnap) {
            batch_free_impl(b);
            set_error("batch_create: cannot copy the cost model");
            return FCFC_EHIP;
        }
        b->kcells = (float)(p->rprune / g.side);
        FCFC_HIP(hipStreamSynchronize(st));
    }
#undef BA
    // pair keys (pair << 6 | cost key) sort in whole bytes; the end key is above them all
    b->sort_bits = 8;
    while (((uint64_t)npairs << 6) >= ((uint64_t)1 << b->sort_bits)) b->sort_bits += 8;
    b->key_last = (uint32_t)(((uint64_t)1 << b->sort_bits) - 1);
    CountArgs& a = b->L.a;
    (void)bind_tables(b->L, b->tab, a);
    a.posA = b->pos32;
    a.absA = b->abs32;
    a.p64A = b->pos64;
    a.wA = b->weighted ? b->w : nullptr;
    a.posB = b->pos32;
    a.p64B = b->pos64;
    a.wB = a.wA;
    a.xstep = key_xstep(g, b->xbits);
    a.items = b->items2;
    a.nitems_dev = &b->ctr[1];
    a.cursor = &b->ctr[2];
    a.out_counts = b->counts;
    a.out_w = b->weighted ? b->wacc : nullptr;
    a.stats = b->kstats;
    a.times = nullptr;
    if (b->weighted) set_weight(a, b->S, b->wmax * b->wmax);
    a.nchunks_dev = &b->ctr[3];
    a.chunk_cursor = &b->ctr[4];
    a.chunk_prefix = b->chunk_prefix;
    a.cat_order = b->pair_order;
    a.cat_items = b->pair_items;
    a.ncat = npairs;
    // A workgroup takes chunks of 32 items per wavefront and waits for its
    // slowest wave at the end of each; measured on MI355X, 8 lost 6 % to those
    // waits and 128 or more left long tails (few chunks per pair).
    const int per_wave = (p->tune.batch_chunk >= 1 && p->tune.batch_chunk <= 1024) ? p->tune.batch_chunk : 32;
    a.chunk_items = std::max(16, b->L.waves * per_wave);
    b->host_args.resize(sizeof(CountArgs));
    memcpy(b->host_args.data(), &a, sizeof(CountArgs));
    FCFC_HIP(hipMemcpy(b->args_dev, b->host_args.data(), sizeof(CountArgs), hipMemcpyHostToDevice));
    b->nblk = grid_blocks(b->L, b->items_cap);
    *out = b;
    return FCFC_OK;
}

fcfc_status batch_run_impl(BatchImpl* b, int64_t* d_counts, double* d_wcounts, bool use_graph, hipStream_t st) {
    Plan* p = b->plan;
    if (d_wcounts && !b->weighted) {
        set_error("batch_run: weighted counts requested but the catalogues have no weights");
        return FCFC_EINVAL;
    }
    if (use_graph) {
        if (!b->gexec) {
            if (!b->cap) FCFC_HIP(hipStreamCreateWithFlags(&b->cap, hipStreamNonBlocking));
            FCFC_HIP(hipStreamSynchronize(st));
            FCFC_HIP(hipStreamBeginCapture(b->cap, hipStreamCaptureModeThreadLocal));
            batch_enqueue_front(b, b->cap);
            batch_enqueue_back(b, b->cap);
            hipGraph_t g = nullptr;
            FCFC_HIP(hipStreamEndCapture(b->cap, &g));
            b->graph = g;
            FCFC_HIP(hipGraphInstantiate(&b->gexec, b->graph, nullptr, nullptr, 0));
        }
        FCFC_HIP(hipEventRecord(b->ev0, st));
        FCFC_HIP(hipGraphLaunch(b->gexec, st));
        FCFC_HIP(hipEventRecord(b->ev1, st));
    } else {
        FCFC_HIP(hipEventRecord(b->ev0, st));
        batch_enqueue_front(b, st);
        batch_enqueue_back(b, st);
        FCFC_HIP(hipEventRecord(b->ev1, st));
    }
    const size_t nbytes = (size_t)b->npairs * p->nbins * 8;
    FCFC_HIP(hipMemcpyAsync(d_counts, b->counts, nbytes, hipMemcpyDeviceToDevice, st));
    if (d_wcounts) FCFC_HIP(hipMemcpyAsync(d_wcounts, b->wout, nbytes, hipMemcpyDeviceToDevice, st));
    return FCFC_OK;
}

fcfc_status batch_check_impl(BatchImpl* b, hipStream_t st, uint32_t* nitems, float* ms) {
    uint32_t h[6];
    FCFC_HIP(hipMemcpyAsync(h, b->ctr, 24, hipMemcpyDeviceToHost, st));
    FCFC_HIP(hipStreamSynchronize(st));
    if (nitems) *nitems = h[1];
    if (ms && hipEventElapsedTime(ms, b->ev0, b->ev1) != hipSuccess) *ms = -1.f;
    if (h[5]) {
        set_error("batch: the work list outgrew the capacity sized at creation (catalogue contents changed)");
        return FCFC_ERANGE;
    }
    return FCFC_OK;
}

fcfc_status batch_stats_impl(BatchImpl* b, hipStream_t st, int64_t out[3]) {
    unsigned long long h[8];
    FCFC_HIP(hipMemcpyAsync(h, b->kstats, 64, hipMemcpyDeviceToHost, st));
    FCFC_HIP(hipStreamSynchronize(st));
    out[0] = (int64_t)h[0];
    out[1] = (int64_t)h[1];
    out[2] = (int64_t)h[6];
    return FCFC_OK;
}

}  // namespace fcfc

using namespace fcfc;

extern "C" fcfc_status fcfc_plan_computed(fcfc_plan_t plan, fcfc_computed* out) {
    clear_error();
    const Plan* p = (const Plan*)plan;
    if (!p || !out) return FCFC_EINVAL;
    if (!p->numerics_ready) {
        set_error("plan_computed: the grid is not fixed yet (set or fit the bounds first)");
        return FCFC_ESTATE;
    }
    CountArgs a;
    memset(&a, 0, sizeof(a));
    set_linear(p, a);
    fcfc_computed c{};
    if (a.lin) {
        set_mu(p, true, a);
        set_filter(p, a);
        c.uniform = 1;
        c.zero2 = a.zero2;
        c.scale1 = a.l1c;
        c.offset1 = a.l1o;
        c.tol1 = a.l1t;
        c.tol1_abs = p->kind == FCFC_BIN_SPERP_PI && p->los == FCFC_LOS_MIDPOINT ? a.l1a : 0.0f;
        c.scale2 = a.l2c;
        c.offset2 = a.l2o;
        c.tol2 = a.l2t;
        c.mu_n = a.mu_c;
        c.mu_tolA = a.tolA;
        c.mu_tolC = a.tolC;
        c.reach = a.f_reach;
        c.e_unit = a.e_unit;
    }
    *out = c;
    return FCFC_OK;
}
