// count_kernel.h -- the persistent pair-counting kernel.
//
// Each wavefront pulls work items (A tile x B row piece) from a global
// cursor and counts them 64 A points at a time.  B points stream past, 64 per
// load; those within reach of the box around the A points are staged in LDS,
// and the matrix cores give the squared separations of 16 of them with the 64
// A points at a time (FP32), from which the pairs in range are compacted into
// a queue.  Per queued pair, one per lane: FP32 displacement and squared
// separation, its bin (computed from the hardware reciprocal square root for
// uniform edges, else from the squared-separation look-up table in LDS of
// Sect. 3.2.3; hot entries resolve by comparison against the FP32 band ends,
// the reverse traversal of Sect. 3.2.1), mu from the same reciprocal square
// root, and an LDS atomic into the workgroup's private histogram
// (Sect. 4.1.2: private histograms instead of conflicting scatters).  Pairs
// inside an error band are queued per wave in LDS and re-evaluated 64 at a
// time with the FP64 definition from the sorted FP64 coordinates.  The
// workgroup histograms are merged into the global int64 (and exact 128-bit
// weighted) accumulators with global atomics.
#pragma once

#include "internal.h"

namespace fcfc {

// Wave-uniform reads (items, leaf origins) go through the constant address
// space so that they become scalar loads; those arrays are never written while
// the kernel runs.
#if defined(__HIP_DEVICE_COMPILE__)
#define FCFC_CONST __attribute__((address_space(4)))
#else
#define FCFC_CONST
#endif
__device__ inline uint32_t ldc_u32(const uint32_t* p, uint32_t i) { return ((const uint32_t FCFC_CONST*)p)[i]; }
__device__ inline int4 ldc_i4(const int4* p, uint32_t i) {
    const int FCFC_CONST* q = (const int FCFC_CONST*)p + 4 * (size_t)i;
    return make_int4(q[0], q[1], q[2], q[3]);
}
__device__ inline Item ldc_item(const Item* p, uint32_t i) {
    const uint32_t FCFC_CONST* q = (const uint32_t FCFC_CONST*)p + 8 * (size_t)i;
    Item it;
    it.a_begin = q[0];
    it.b_begin = q[1];
    it.b_end = q[2];
    it.a_count = q[3];
    it.meta = q[4];
    it.cost = q[5];
    it.tile = q[6];
    return it;
}

enum { COUNT_SINGLE = 0, COUNT_BATCH = 1, COUNT_TREE = 2 };
constexpr int CT_MAX = 1024;        // threads per workgroup (16 waves: 4 per SIMD, one workgroup per CU)
constexpr int QCAP = 320;           // queue entries per wave: 63 waiting plus a step of 256 candidates
// recheck entries per wave: RB_FLUSH - 1 waiting plus the up to 64 of one
// binning pass (rechecks are rare; a small buffer leaves LDS for more waves)
constexpr int RB_FLUSH = 32;
constexpr int RB_CAP = RB_FLUSH + 64;
constexpr int ASTAGE = 64;          // staged A points per wave
constexpr int BSTAGE = 80;          // staged B points per wave: 15 waiting plus a batch of 64
// LDS of one wave: staged A and B points, absolute A points (mid-point),
// recheck entries (item, pair), queue, the staged points' weights.  (Weights
// read from memory for every pair, as it came from the queue, left the few
// waves of a weighted count waiting on them: on MI355X 1M weighted points in
// 4,000 bins ran 5.61 -> 5.08 ms, a weighted survey of 200k x 4M 76.6 -> 72.5.)
__host__ __device__ constexpr int wave_lds_bytes(bool mid, bool weighted) {
    return (ASTAGE + BSTAGE + (mid ? ASTAGE : 0)) * 16 + RB_CAP * 8 + QCAP * 2 + (weighted ? (ASTAGE + BSTAGE) * 8 : 0);
}
constexpr uint32_t OFF_SA = 0, OFF_SB = ASTAGE * 16, OFF_SABS = (ASTAGE + BSTAGE) * 16;
constexpr uint32_t OFF_SWA(bool mid) { return (uint32_t)wave_lds_bytes(mid, false); }
constexpr uint32_t OFF_SWB(bool mid) { return OFF_SWA(mid) + ASTAGE * 8; }
// A wavefront empties the LDS histograms into the outputs after claiming
// 2^26 candidate pairs since it last did (fcfc_tuning.flush_log2 lowers it).
constexpr int FLUSH_LOG2_MAX = 26;

// Format of the exact weighted sums in LDS (add_weight).
struct WeightFmt {
    double scale, mul, bias;  // 2^(S - k), 2^k, 2^(k - 1)
    unsigned long long one;   // 2^cs
    int k, cs;
    uint32_t limit;           // pairs a wave tests before it empties the words
};

struct CountArgs {
    const float4* posA;
    const float4* absA;
    const double* p64A;
    const double* wA;
    const float4* posB;
    const double* p64B;
    const double* wB;
    const Item* items;
    const uint32_t* nitems_dev;
    uint32_t* cursor;
    const int16_t* lut1;
    const int16_t* lut2;
    const float2* band1;  // (lo_k, hi_k) for k = 0..n1, then (+inf, +inf)
    const float2* band2;
    const double* E1;    // FP64 squared edges
    const double* E2;
    unsigned long long* out_counts;
    unsigned long long* out_w;  // 2 per bin: low, high 64 bits of a signed 128-bit sum
    unsigned long long* stats;  // [0] candidates [1] rechecks [5] bad prediction [6] early merges
    uint32_t* times;            // per item duration (wall clock ticks) or null
    int nlut1, nlut2;
    float scale1, scale2, vmax1, vmax2;
    int n1, n2, nbins;
    int nx;
    float side32;
    // tree counts: lattice origins of the A and B leaves (units of tree_q),
    // points per leaf and B leaves
    const int4* leaf_orgA;
    const int4* leaf_orgB;
    float tree_q;
    uint32_t tree_leaf, tree_nleafB;
    double L, halfL;
    // candidate filter (set_filter): squared separation (its transverse part
    // for (s_perp, pi)), squared reach from the box of the A points, second
    // axis, and the margins
    float f_t2, f_cull2, f_u, f_reach, f_slack, f_uslack, f_uerr, f_ts;
    float f_ext;  // tree: largest leaf-local coordinate
    float f_sig, f_inv, f_inv2;  // the filter's unit: a power of two, its inverse and that squared
    // uniform edges: x = s l1c + l1o (and |pi| l2c + l2o) is the bin plus a
    // fraction, good to l1a / s + l1t (l2t)
    int lin;
    float l1c, l1o, l1a, l1t, l2c, l2o, l2t;
    int zero2;  // the second axis starts at 0
    float e_unit;  // u over the error of one displacement component
    float xstep;   // a row's points are sorted by x to this
    float mu_n, mu_c, tolA, tolC;  // mu_c: what mu n2 is formed with (set_mu)
    int mu_top_closed;
    WeightFmt wf;
    int copies;
    unsigned long long flush_pairs;     // a wave merges after claiming this many pairs
    uint32_t shard_count, shard_index;  // this launch takes items shard_index, + shard_count, ...
    // batched mode: chunks of items per output histogram (one per catalogue pair)
    const uint32_t* nchunks_dev;
    uint32_t* chunk_cursor;
    const uint32_t* chunk_prefix;  // ncat + 1, in histogram order
    const uint32_t* cat_order;     // histogram index at each order position
    const uint32_t* cat_items;     // ncat + 1: items of histogram c are [cat_items[c], cat_items[c+1])
    int ncat;                      // histograms
    int chunk_items;
    // LDS layout (bytes)
    int off_lut1, off_lut2, off_band1, off_band2, off_hist, off_whist, off_wave, off_misc, lds_bytes;
};

// The arguments live in device memory and are read through the constant
// address space (scalar loads); a by-value kernel argument would be copied to
// scratch as soon as a helper takes its address.
typedef const CountArgs FCFC_CONST& ArgsRef;

struct Smem {
    const int16_t* lut1;
    const int16_t* lut2;
    const float2* band1;
    const float2* band2;
    uint32_t* hist;
    uint32_t wl, wstride;    // weighted words: LDS address of the first, bytes to the second word of a bin
    // this wave's
    uint32_t wbase;   // LDS byte address of its part
    uint16_t* q;      // queue of pairs: b_slot << 6 | a_slot
    uint32_t qbase;   // its LDS byte address
    uint32_t* rb;     // recheck entries (item, (b - b_begin) << 7 | a - a_begin)
    float4* sa;       // staged A points
    float4* sb;       // staged B points
    double *swa, *swb;  // weights of the staged points
    float4* sabs;     // twice the A points in absolute FP32 (mid-point line of sight)
    unsigned long long* misc;
};

// ---------------------------------------------------------------------------
// FP64 definition (independent of the FP32 path): bins of one pair from the
// sorted FP64 coordinates.  Contraction is disabled for the whole library, so
// each product and sum below rounds separately, in the order written.
// Returns the flat bin or -1.  For a periodic box the item's image shift must
// be the minimum image of b as seen from a, otherwise the pair belongs to
// another item and -1 is returned.
// ---------------------------------------------------------------------------
__device__ inline int upper_edge_count(const double* __restrict__ E, int n, double v) {
    // number of edges E[0..n] with E[k] <= v (binary search)
    int lo = 0, hi = n + 1;
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (E[mid] <= v) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

template <int KIND, int LOS>
__device__ int exact_bin(ArgsRef a, double ax, double ay, double az, double bx, double by, double bz,
                         int sx, int sy, int sz) {
    double dx = bx - ax;
    double dy = by - ay;
    double dz = bz - az;
    if (a.L > 0.0) {
        int cx = 0, cy = 0, cz = 0;
        if (dx > a.halfL) { dx -= a.L; cx = -1; } else if (dx < -a.halfL) { dx += a.L; cx = 1; }
        if (dy > a.halfL) { dy -= a.L; cy = -1; } else if (dy < -a.halfL) { dy += a.L; cy = 1; }
        if (dz > a.halfL) { dz -= a.L; cz = -1; } else if (dz < -a.halfL) { dz += a.L; cz = 1; }
        if (cx != sx || cy != sy || cz != sz) return -1;
    }
    double xx = dx * dx;
    double yy = dy * dy;
    double zz = dz * dz;
    double d2 = (xx + yy) + zz;
    double pi2 = 0.0;
    if (KIND != FCFC_BIN_S) {
        if (LOS == FCFC_LOS_Z) {
            pi2 = zz;
        } else {
            double lx = ax + bx;
            double ly = ay + by;
            double lz = az + bz;
            double t1 = dx * lx;
            double t2 = dy * ly;
            double t3 = dz * lz;
            double dot = (t1 + t2) + t3;
            double q1 = lx * lx;
            double q2 = ly * ly;
            double q3 = lz * lz;
            double ll = (q1 + q2) + q3;
            double dd = dot * dot;
            pi2 = (ll > 0.0) ? dd / ll : 0.0;
        }
    }
    if (KIND == FCFC_BIN_S || KIND == FCFC_BIN_S_MU) {
        int c = upper_edge_count(a.E1, a.n1, d2);
        if (c < 1 || c > a.n1) return -1;
        int k = c - 1;
        if (KIND == FCFC_BIN_S) return k;
        int j;
        if (d2 == 0.0) {
            j = 0;  // mu = 0; the first mu edge is 0
        } else {
            // largest j in [0, n2] with (j/n2)^2 * d2 <= pi2
            int lo = 0, hi = a.n2 + 1;
            while (lo < hi) {
                int mid = (lo + hi) >> 1;
                double m = (double)mid / (double)a.n2;
                double M = m * m;
                if (M * d2 <= pi2) lo = mid + 1;
                else hi = mid;
            }
            j = lo - 1;  // >= 0 since M_0 = 0
            if (j == a.n2) {
                if (!a.mu_top_closed) return -1;
                j = a.n2 - 1;
            }
        }
        return k * a.n2 + j;
    }
    double sp2;
    if (LOS == FCFC_LOS_Z) {
        sp2 = xx + yy;
    } else {
        sp2 = d2 - pi2;
        if (sp2 < 0.0) sp2 = 0.0;
    }
    int c1 = upper_edge_count(a.E1, a.n1, sp2);
    if (c1 < 1 || c1 > a.n1) return -1;
    int c2 = upper_edge_count(a.E2, a.n2, pi2);
    if (c2 < 1 || c2 > a.n2) return -1;
    return (c1 - 1) * a.n2 + (c2 - 1);
}

// ---------------------------------------------------------------------------
// FP32 look-up with bands: returns bin (>= 0), -1 (out of range) or sets amb.
// ---------------------------------------------------------------------------
__device__ inline int lut_entry(const int16_t* __restrict__ lut, float scale, float v) {
    return (int)lut[(uint32_t)(v * scale)];
}
// A clean entry (>= -1) is the bin itself, -1 meaning out of range.  A hot
// entry (<= -2) holds -2 - k, k the first edge whose band meets the entry (the
// edges below k lie wholly below the entry).  Most hot entries meet one band:
// v is then placed by band k and the start of band k + 1, read together; when
// v reaches band k + 1 (several edges in one entry) the walk goes on over the
// next bands.  band[k] = (lo_k, hi_k), band[n + 1] = (+inf, +inf).  Returns the
// bin, -1 (out of range) or -2 (v inside a band: the pair needs the FP64
// recheck).
__device__ inline int lut_hot_bin(const float2* __restrict__ band, int n, int e, float v) {
    int k = -2 - e;
    const float2 b0 = band[k];
    const float lo1 = band[k + 1].x;
    if (v < b0.x) return k - 1;
    if (v < b0.y) return -2;
    if (v < lo1) return k < n ? k : -1;
    for (k = k + 1; k <= n; k++) {
        const float2 b = band[k];
        if (v >= b.y) continue;
        if (v >= b.x) return -2;
        break;
    }
    return (k >= 1 && k <= n) ? k - 1 : -1;
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

// LDS by byte address
typedef __attribute__((address_space(3))) const uint16_t LdsU16;
typedef __attribute__((address_space(3))) const f32x4 LdsF4;
typedef __attribute__((address_space(3))) uint32_t LdsU32;
__device__ inline uint32_t lds_u16(uint32_t at) { return *(LdsU16*)at; }
__device__ inline f32x4 lds_f4(uint32_t at) { return *(LdsF4*)at; }
__device__ inline double lds_f64(uint32_t at) { return *(__attribute__((address_space(3))) const double*)at; }
__device__ inline float lds_f1(uint32_t at) { return *(__attribute__((address_space(3))) const float*)at; }
__device__ inline void lds_inc(uint32_t at) {
    __hip_atomic_fetch_add((LdsU32*)at, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
template <typename T>
__device__ inline uint32_t lds_addr(T* p) { return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) T*)p; }
typedef __attribute__((address_space(3))) unsigned long long LdsU64;
__device__ inline void lds_add_u64(uint32_t at, unsigned long long v) {
    __hip_atomic_fetch_add((LdsU64*)at, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ inline unsigned long long lds_exch_u64(uint32_t at) {
    return __hip_atomic_exchange((LdsU64*)at, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Kernel constants kept in registers.
struct KConst {
    float scale1, scale2, vmax1, vmax2, mu_n, mu_nm1, tolA, tolC, side32;
    int lin;
    float l1c, l1o, l1a, l1t, l2c, l2o, l2t;  // uniform edges (CountArgs)
    int zero2;
    float tolC_v;  // tolC held in a vector register (an fma takes one scalar operand)
    int n1, n2, nbins, nx, copies;
    WeightFmt wf;
};

// largest integer at or below x (any integer for a NaN) in one instruction
__device__ inline int floor_i(float x) {
    int r;
    __asm__("v_cvt_flr_i32_f32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}

// With computed bins mu n2 is formed with n2 times one minus this, more than the
// rounding of mu (two or three reciprocal square roots of 4.8e-7 at most and a
// few products, 0.8e-6 along z and 1.6e-6 to the mid-point), so that mu = 1 needs
// no clamp; the mu bands are wider by as much.  (With the bins rounded down
// instead of truncated and shifted: on MI355X 16 mocks of 100,000 to 500,000
// points 36.5 -> 35.7 ms.)
__host__ __device__ constexpr float mu_shrink(bool mid) { return mid ? 0x1p-18f : 0x1p-19f; }

// Add a pair of weight p to bin `flat` of a weighted count.  p 2^S is an
// integer q (the host chose S), |q| <= 2^qb; with q = i 2^k + r, |r| <= 2^(k-1),
// the bin holds two 64-bit words,
//   sum of (r + 2^(k-1)), from bit cs on the number of pairs, and
//   sum of i (signed),
// which stay exact for 2^N pairs: (qb - k) + N <= 62, cs = k + N + 1 and
// cs + N + 1 <= 64 (set_weight; N is 20 to 23, and a wave empties the
// workgroup's words in time).  i comes out of the low bits of t + 1.5 2^52,
// t = p 2^(S-k), which rounds t to an integer; every step is exact in FP64.
// Two LDS additions a pair instead of three, and 16 bytes a bin instead of 20:
// the additions on random bins collide (half of the LDS cycles of a weighted
// count).  On MI355X a weighted survey of 200k x 4M ran 80.4 -> 75.4 ms; 1M
// weighted points in 4,000 bins gained nothing, where vector instructions bound
// the kernel.  With the two words side by side, on half as many banks, the
// survey took 79 ms.
__device__ inline void add_weight(const Smem& s, const WeightFmt& f, uint32_t flat, double p) {
    const double magic = 6755399441055744.0;  // 1.5 2^52
    const double t = p * f.scale;
    const double x = t + magic;
    const double r = t - (x - magic);
    const uint32_t lo = (uint32_t)__builtin_fma(r, f.mul, f.bias);
    const unsigned long long hi = (unsigned long long)__double_as_longlong(x) - 0x4338000000000000ull;
    const uint32_t at = s.wl + (flat << 3);
    lds_add_u64(at, f.one + (unsigned long long)lo);
    lds_add_u64(at + s.wstride, hi);
}
// The two words of a bin, taken out: number of pairs, and their sum times 2^S.
__device__ inline uint32_t weight_words(const WeightFmt& f, unsigned long long lo, unsigned long long hi, __int128& sum) {
    const uint32_t n = (uint32_t)(lo >> f.cs);
    const long long rest = (long long)(lo & ((1ull << f.cs) - 1ull)) - ((long long)n << (f.k - 1));
    sum = ((__int128)(long long)hi << f.k) + (__int128)rest;
    return n;
}
__device__ inline void add_out_w(unsigned long long* out, __int128 v) {
    const unsigned long long vlo = (unsigned long long)v;
    unsigned long long vhi = (unsigned long long)(v >> 64);
    const unsigned long long o = atomicAdd(out, vlo);
    if (o + vlo < o) vhi += 1ull;
    if (vhi) atomicAdd(out + 1, vhi);
}

// Re-evaluate `cnt` queued pairs (entries base .. base+cnt-1) in FP64.
template <int KIND, int LOS, bool W>
__device__ __attribute__((always_inline)) inline void process_rechecks(ArgsRef a, const Smem& s, int base, int cnt, int lane,
                                 unsigned long long& nrechk) {
    if (lane < cnt) {
        const uint32_t* e = s.rb + (size_t)(base + lane) * 2;
        const Item* it = a.items + e[0];
        const uint32_t ia = it->a_begin + (e[1] & 127u), ib = it->b_begin + (e[1] >> 7);
        const uint32_t meta = it->meta;
        int sx = (int)((meta >> 16) & 3u) - 1;
        int sy = (int)((meta >> 18) & 3u) - 1;
        int sz = (int)((meta >> 20) & 3u) - 1;
        const double* pa = a.p64A + 3 * (size_t)ia;
        const double* pb = a.p64B + 3 * (size_t)ib;
        int flat = exact_bin<KIND, LOS>(a, pa[0], pa[1], pa[2], pb[0], pb[1], pb[2], sx, sy, sz);
        if (flat >= 0) {
            if (W)
                add_weight(s, a.wf, (uint32_t)flat, a.wA[ia] * a.wB[ib]);
            else
                atomicAdd(&s.hist[flat], 1u);
        }
    }
    nrechk += (unsigned long long)cnt;
}

__device__ inline void wave_sync_lds() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Third word of a raw buffer resource on gfx9-family devices (32-bit data format).
constexpr int BUFFER_RSRC_WORD3 = 0x00020000;

// 16 bytes at byte offset voff + soff of a buffer (zeros past its end).
__device__ inline float4 load_b(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, (int)soff, 0);
    return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
}

__device__ inline uint32_t lane_prefix(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Per-wave context of the current work item: 64 of its A points against its
// B points.
struct WaveCtx {
    uint32_t aslot0;   // position of A slot 0 in the item's A tile (0 or 64)
    uint32_t it;
    int rcount;
    unsigned long long nrechk;
    float t1, t1a, t2, tA, tC;  // tolerances of the computed bins, widened for this tile
};

// Bin `cnt` queued pairs (entries base .. base+cnt-1), one per lane.  An entry
// is b_slot << 6 | a_slot, slots of the staged points.  Staged A points hold
// the cell-local position (y and z moved into the B row's frame) and the cell
// x as a float; staged B points the cell-local position and, in w, the point's
// offset in the item << 11 | cell x (both cell x counted from the tile's first
// cell, plus 64).  The queue holds every pair in range and a few just beyond
// (the filter of process_half is conservative), so the pair is formed here in
// cell-local FP32, the arithmetic the error bands are derived for.
// The common path is branch-free; hot table entries and rechecks take
// wave-uniform branches that are rarely entered.
// Where the edges of every axis are uniform (LIN) the bin is computed, not
// looked up: x = (s - e_0) / ds + 1 from the hardware reciprocal square root,
// its integer part the bin plus one, and a pair within the FP32 error of an
// integer goes to the FP64 recheck.  That takes 7 vector instructions; the
// table takes 8 and an LDS read, and about 15 more whenever one of 64 pairs
// meets an entry with an edge in it, which was more than every second time.
template <int KIND, int LOS, bool W, bool TREE, bool LIN>
__device__ __attribute__((always_inline)) inline void bin_queue(ArgsRef a, const KConst& k, const Smem& s,
                                                                uint32_t hist_l, uint32_t qrow, int cnt, int lane,
                                                                WaveCtx& c) {
    constexpr bool MID = (LOS == FCFC_LOS_MIDPOINT && KIND != FCFC_BIN_S);
    constexpr bool SPI = KIND == FCFC_BIN_SPERP_PI;
    // lanes past the last entry read stale entries (valid slots) and are masked below
    const uint32_t id = lds_u16(qrow + 2u * (uint32_t)lane);
    const uint32_t as = id & 63u;
    uint32_t bs = id >> 6;
    __asm__ volatile("" : "+v"(bs));
    const f32x4 A = lds_f4(s.wbase + OFF_SA + (as << 4));
    const f32x4 B = lds_f4(s.wbase + OFF_SB + (bs << 4));
    const uint32_t bw = __float_as_uint(B.w);
    double wa = 0.0, wb = 0.0;
    if (W) {
        wa = lds_f64(s.wbase + OFF_SWA(MID) + (as << 3));
        wb = lds_f64(s.wbase + OFF_SWB(MID) + (bs << 3));
    }
    float dx, dy, dz;
    if (TREE || LIN) {  // both in the frame of the A points
        dx = B.x - A.x;
    } else {
        const float D = ((float)(bw & 255u) - A.w) * k.side32;
        dx = B.x - (A.x - D);
    }
    dy = B.y - A.y;
    dz = B.z - A.z;
    // Wave masks, each built from ballots of single compares (a ballot of a
    // compare is that compare's lane mask, so no per-lane boolean is formed):
    //   rm: pairs within an FP32 band of an edge (FP64 recheck),
    //   um: pairs binned here (in range, not rechecked).
    const uint64_t vmask = cnt >= 64 ? ~0ull : ((1ull << cnt) - 1ull);
    uint64_t rm, um;
    int flat;
    // (in range is decided by the bins: the filter lets pairs just beyond pass)
    float d2 = 0.f, lsq = 1.f, dot = 0.f;  // line of sight: dot = d.l, lsq = |l|^2
    if (!(SPI && !MID)) d2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
    if (MID) {
        const f32x4 q = lds_f4(s.wbase + OFF_SABS + (as << 4));
        const float lx = q.x + dx, ly = q.y + dy, lz = q.z + dz;
        dot = __builtin_fmaf(dz, lz, __builtin_fmaf(dy, ly, dx * lx));
        lsq = __builtin_fmaf(lz, lz, __builtin_fmaf(ly, ly, lx * lx));
    }
    int b2 = 0;           // second bin
    float b2f = 0.f;      // computed bins: with its fraction
    uint64_t near2 = 0;   // pairs near an edge of the second axis
    uint64_t in2 = ~0ull; // pairs in range of the second axis
    uint64_t sure = 0;    // pairs in range and near no edge of the first axis
    float v1 = d2, rs = 0.f;  // first axis: squared separation, and its reciprocal square root
    if (KIND == FCFC_BIN_S_MU) {
        const float proj_n = MID ? fabsf(dot) * (__builtin_amdgcn_rsqf(lsq) * k.mu_n) : fabsf(dz) * k.mu_n;
        rs = __builtin_amdgcn_rsqf(d2);
        const float mun = proj_n * rs;
        // (with computed bins mu_n is a little below n2, so that mun stays below n2)
        b2 = LIN ? (int)mun : min((int)mun, k.n2 - 1);
        // distance to the nearest interior mu edge (edges 0 and n need no recheck: mu
        // >= 0 always, and mu = 1 belongs to the last bin); not a number at zero
        // separation, which is a recheck too
        const float cr = __builtin_amdgcn_fmed3f(rintf(mun), 1.0f, k.mu_nm1);
        const float tol = LIN ? __builtin_fmaf(c.tA, rs, c.tC) : __builtin_fmaf(k.tolA, rs, k.tolC_v);
        near2 = __builtin_amdgcn_ballot_w64(!(fabsf(mun - cr) >= tol));
    }
    if (LIN) {
        if (SPI) {
            float p;  // |pi|
            if (MID) {
                p = fabsf(dot) * __builtin_amdgcn_rsqf(lsq);
                v1 = fmaxf(__builtin_fmaf(-p, p, d2), 0.0f);
            } else {
                p = fabsf(dz);
                v1 = __builtin_fmaf(dy, dy, dx * dx);
            }
            b2f = __builtin_fmaf(p, k.l2c, k.l2o);
            b2 = floor_i(b2f);
            near2 = __builtin_amdgcn_ballot_w64(!(fabsf(b2f - rintf(b2f)) >= c.t2));
            in2 = __builtin_amdgcn_ballot_w64((uint32_t)b2 < (uint32_t)k.n2);
        }
        if (KIND != FCFC_BIN_S_MU) rs = __builtin_amdgcn_rsqf(v1);
        const float x1 = __builtin_fmaf(v1 * rs, k.l1c, k.l1o);
        const int b1 = floor_i(x1);
        // |s32 - s| is bounded by the displacement's error; the mid-point s_perp^2 is a
        // difference, good to an absolute error: that over s_perp
        const float tol1 = SPI && MID ? __builtin_fmaf(c.t1a, rs, c.t1) : c.t1;
        const uint64_t near1 = __builtin_amdgcn_ballot_w64(!(fabsf(x1 - rintf(x1)) >= tol1));
        rm = (near1 | near2) & vmask;
        const uint64_t in = __builtin_amdgcn_ballot_w64((uint32_t)b1 < (uint32_t)k.n1) & in2 & vmask;
        um = in & ~rm;
        if (SPI && !MID) sure = in & ~near1;
        flat = KIND == FCFC_BIN_S ? b1 : (int)__umul24((uint32_t)b1, (uint32_t)k.n2) + b2;
    } else if (!SPI) {
        const float d2c = __builtin_amdgcn_fmed3f(d2, 0.0f, k.vmax1);  // at vmax the table says out of range
        int sb = lut_entry(s.lut1, k.scale1, d2c);
        if (sb < -1) sb = lut_hot_bin(s.band1, k.n1, sb, d2c);
        rm = (__builtin_amdgcn_ballot_w64(sb == -2) | (near2 & __builtin_amdgcn_ballot_w64(d2 < k.vmax1))) & vmask;
        um = __builtin_amdgcn_ballot_w64(sb >= 0) & vmask & ~rm;
        flat = KIND == FCFC_BIN_S ? sb : (int)__umul24((uint32_t)sb, (uint32_t)k.n2) + b2;
    } else {
        float sp2, pi2;
        if (!MID) {
            sp2 = __builtin_fmaf(dy, dy, dx * dx);
            pi2 = dz * dz;
        } else {
            pi2 = (dot * dot) * __builtin_amdgcn_rcpf(lsq);
            sp2 = fmaxf(d2 - pi2, 0.0f);
        }
        // beyond a table's top band end the pair is certainly out of range
        const uint64_t inm =
            __builtin_amdgcn_ballot_w64(sp2 < k.vmax1) & __builtin_amdgcn_ballot_w64(pi2 < k.vmax2) & vmask;
        const bool inr = __builtin_amdgcn_inverse_ballot_w64(inm);
        const float sp2c = inr ? sp2 : 0.0f;
        const float pi2c = inr ? pi2 : 0.0f;
        int b1 = lut_entry(s.lut1, k.scale1, sp2c);
        b2 = lut_entry(s.lut2, k.scale2, pi2c);
        if (b1 < -1) b1 = lut_hot_bin(s.band1, k.n1, b1, sp2c);
        if (b2 < -1) b2 = lut_hot_bin(s.band2, k.n2, b2, pi2c);
        rm = (__builtin_amdgcn_ballot_w64(b1 == -2) | __builtin_amdgcn_ballot_w64(b2 == -2)) & inm;
        um = __builtin_amdgcn_ballot_w64(b1 >= 0) & __builtin_amdgcn_ballot_w64(b2 >= 0) & inm & ~rm;
        flat = (int)__umul24((uint32_t)b1, (uint32_t)k.n2) + b2;
    }
    if (__builtin_amdgcn_inverse_ballot_w64(um)) {
        if (W)
            add_weight(s, k.wf, (uint32_t)flat, wa * wb);
        else
            lds_inc(hist_l + ((uint32_t)flat << 2));
    }
    uint64_t m = rm;
    if (m) {
        if (LIN && SPI && !MID && k.zero2) {
            // Nothing lies below an edge at 0: a pair near that one only is certain.
            // (Without this a catalogue in a plane rechecked every pair for its pi = 0:
            // MI355X, 60,000 points in one plane, 4.11 -> 1.02 ms; 400,000 points at
            // random 1.14 ms with and without.)
            const uint64_t z = m & sure & __builtin_amdgcn_ballot_w64(b2f < 1.0f - c.t2);
            if (__builtin_amdgcn_inverse_ballot_w64(z)) {
                if (W)
                    add_weight(s, k.wf, (uint32_t)flat, wa * wb);
                else
                    lds_inc(hist_l + ((uint32_t)flat << 2));
            }
            m &= ~z;
        }
        const int pos = c.rcount + (int)lane_prefix(m);
        if (__builtin_amdgcn_inverse_ballot_w64(m)) {
            uint32_t* r = s.rb + (size_t)pos * 2;
            r[0] = c.it;
            r[1] = ((bw >> 11) << 7) | (c.aslot0 + as);
        }
        c.rcount += (int)__popcll(m);
        if (c.rcount >= RB_FLUSH) {
            const int n = c.rcount < 64 ? c.rcount : 64;
            wave_sync_lds();
            process_rechecks<KIND, LOS, W>(a, s, c.rcount - n, n, lane, c.nrechk);
            wave_sync_lds();
            c.rcount -= n;
        }
    }
}

// Wave-wide minimum and maximum (valid in every lane) by DPP row shifts and
// row broadcasts.
template <int CTRL, int ROWS>
__device__ inline float dpp_from(float v) {
    return __int_as_float(
        __builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), CTRL, ROWS, 0xf, false));
}
__device__ inline float wave_min_f(float v) {
    v = fminf(v, dpp_from<0x111, 0xf>(v));
    v = fminf(v, dpp_from<0x112, 0xf>(v));
    v = fminf(v, dpp_from<0x114, 0xf>(v));
    v = fminf(v, dpp_from<0x118, 0xf>(v));
    v = fminf(v, dpp_from<0x142, 0xa>(v));
    v = fminf(v, dpp_from<0x143, 0xc>(v));
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ inline float wave_max_f(float v) { return -wave_min_f(-v); }
__device__ inline float uniform_f(float v) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// Positions of the work list held by a workgroup in LDS: one 64-bit word
// (end << 32 | next) that a wave takes from with one addition, refilled by
// whichever wave finds it empty and gets the lock.  The holder waits for
// nothing but its own atomics, so every other wave's wait ends.
struct WorkClaim {
    unsigned long long* word;
    uint32_t *lk, *done;
    __device__ explicit WorkClaim(unsigned long long* misc)
        : word(misc), lk((uint32_t*)(misc + 1)), done((uint32_t*)(misc + 1) + 1) {}
    __device__ bool take(uint32_t& pos) {
        if (empty()) return false;
        const unsigned long long v =
            __hip_atomic_fetch_add(word, 1ull, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
        if ((uint32_t)v >= (uint32_t)(v >> 32)) return false;
        pos = (uint32_t)v;
        return true;
    }
    __device__ bool empty() const {
        const unsigned long long v = __hip_atomic_load(word, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
        return (uint32_t)v >= (uint32_t)(v >> 32);
    }
    __device__ uint32_t end() const {
        return (uint32_t)(__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) >> 32);
    }
    __device__ bool drained() const {
        return __hip_atomic_load(done, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) != 0u && empty();
    }
    __device__ bool lock() {
        return __hip_atomic_exchange(lk, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP) == 0u;
    }
    __device__ void unlock() { __hip_atomic_store(lk, 0u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP); }
    // positions [at, end) of a list of n: none are left when at reaches n
    __device__ void refill(uint32_t at, uint32_t end, uint32_t n) {
        if (at < n)
            __hip_atomic_store(word, (unsigned long long)end << 32 | at, __ATOMIC_RELEASE,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
        else
            __hip_atomic_store(done, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
};


// Append `id` of the lanes in the mask to the queue whose end is LDS byte
// address `end` (wave-uniform).  The store runs under the mask itself, set
// and restored around it (every lane of the wave is active here): a branch
// around an empty store costs more than the store.
__device__ inline void queue_append(uint32_t& end, uint64_t in, uint32_t id) {
    const uint32_t pre = __builtin_amdgcn_mbcnt_hi((uint32_t)(in >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)in, 0u));
    const uint32_t at = (pre << 1) + end;
    __asm__ volatile(
        "s_mov_b64 exec, %2\n\t"
        "ds_write_b16 %0, %1\n\t"
        "s_mov_b64 exec, -1"
        :
        : "v"(at), "v"(id), "s"(in)
        : "memory");
    end += 2u * (uint32_t)__popcll(in);
    __asm__ volatile("" : "+s"(end));  // (kept as one running address)
}

// Registers: unweighted s and (s, mu) counts along z are held to 64 VGPRs,
// eight waves per SIMD in two 16-wave workgroups (on MI355X a mock of 200,003
// points ran 1.62 ms against 1.70 ms at six; the spills this costs sit in the
// per-item code), other unweighted ones to 80, six waves in two 12-wave
// workgroups.  (72 VGPRs and two 14-wave workgroups do not pay: both
// workgroups' odd waves go to the same SIMDs, and only one fits.)  Weighted
// counts are held to 16 waves per CU by their LDS sums and keep the registers.
// MODE: COUNT_SINGLE (one grid count), COUNT_BATCH (a stacked build's pair
// list) or COUNT_TREE (a count over k-d tree leaves).
template <int KIND, int LOS, bool AUTO, bool W, int MODE, bool LIN>
__global__ __launch_bounds__(CT_MAX) __attribute__((amdgpu_waves_per_eu(W ? 4 : (!LOS && KIND != FCFC_BIN_SPERP_PI ? 8 : 6))))
void k_count(const CountArgs* argp) {
    constexpr bool BATCH = MODE == COUNT_BATCH;
    constexpr bool TREE = MODE == COUNT_TREE;
    constexpr bool MID = (LOS == FCFC_LOS_MIDPOINT && KIND != FCFC_BIN_S);
    constexpr bool SPI = KIND == FCFC_BIN_SPERP_PI;
    ArgsRef a = *(const CountArgs FCFC_CONST*)argp;
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x;
    const int nthr = blockDim.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    Smem s;
    s.lut1 = (const int16_t*)(smem + a.off_lut1);
    s.lut2 = (const int16_t*)(smem + a.off_lut2);
    s.band1 = (const float2*)(smem + a.off_band1);
    s.band2 = (const float2*)(smem + a.off_band2);
    s.hist = (uint32_t*)(smem + a.off_hist);
    s.wl = lds_addr(smem + a.off_whist);
    s.wstride = 8u * (uint32_t)a.nbins;
    {
        unsigned char* pw = smem + a.off_wave + (size_t)wave * wave_lds_bytes(MID, W);
        s.wbase = lds_addr(pw);
        s.sa = (float4*)pw;
        pw += ASTAGE * 16;
        s.sb = (float4*)pw;
        pw += BSTAGE * 16;
        s.sabs = (float4*)pw;
        if (MID) pw += ASTAGE * 16;
        s.rb = (uint32_t*)pw;
        pw += RB_CAP * 8;
        s.q = (uint16_t*)pw;
        pw += QCAP * 2;
        s.swa = (double*)pw;
        s.swb = s.swa + ASTAGE;
        s.qbase = lds_addr(s.q);
        for (int i = lane; i < QCAP / 2; i += 64) ((uint32_t*)s.q)[i] = 0u;
    }
    s.misc = (unsigned long long*)(smem + a.off_misc);

    // stage tables, clear histograms
    {
        uint32_t* d = (uint32_t*)(smem + a.off_lut1);
        const uint32_t* src = (const uint32_t*)a.lut1;
        for (int i = tid; i < (a.nlut1 + 1) / 2; i += nthr) d[i] = src[i];
        if (KIND == FCFC_BIN_SPERP_PI) {
            d = (uint32_t*)(smem + a.off_lut2);
            src = (const uint32_t*)a.lut2;
            for (int i = tid; i < (a.nlut2 + 1) / 2; i += nthr) d[i] = src[i];
        }
        float2* b1 = (float2*)(smem + a.off_band1);
        for (int i = tid; i < a.n1 + 2; i += nthr) b1[i] = a.band1[i];
        if (KIND == FCFC_BIN_SPERP_PI) {
            float2* b2 = (float2*)(smem + a.off_band2);
            for (int i = tid; i < a.n2 + 2; i += nthr) b2[i] = a.band2[i];
        }
        if (W)
            for (int i = tid; i < 2 * a.nbins; i += nthr) ((unsigned long long*)(smem + a.off_whist))[i] = 0ull;
        else
            for (int i = tid; i < a.nbins * a.copies; i += nthr) s.hist[i] = 0u;
        if (tid < 4) s.misc[tid] = 0ull;
    }
    __syncthreads();

    KConst k;
    k.scale1 = a.scale1;
    k.scale2 = a.scale2;
    k.vmax1 = a.vmax1;
    k.vmax2 = a.vmax2;
    k.mu_n = a.mu_c;
    k.mu_nm1 = a.mu_n - 1.0f;
    k.tolA = a.tolA;
    k.tolC = a.tolC;
    k.tolC_v = k.tolC;
    __asm__ volatile("" : "+v"(k.tolC_v));
    k.side32 = a.side32;
    k.n1 = a.n1;
    k.n2 = a.n2;
    k.nbins = a.nbins;
    k.nx = a.nx;
    k.copies = a.copies;
    if (W) k.wf = a.wf;
    // (kept in registers: the compiler would load them again for every row)
    k.l1c = a.l1c;
    k.l1o = a.l1o;
    k.l1a = a.l1a;
    k.l1t = a.l1t;
    k.l2c = a.l2c;
    k.l2o = a.l2o;
    k.l2t = a.l2t;
    k.zero2 = a.zero2;
    __asm__ volatile("" : "+s"(k.side32));
    if (LIN) __asm__ volatile("" : "+s"(k.l1c), "+v"(k.l1o), "+s"(k.l1t));
    if (!LIN) __asm__ volatile("" : "+s"(k.scale1), "+s"(k.vmax1));
    if (KIND == FCFC_BIN_S_MU) __asm__ volatile("" : "+s"(k.mu_n), "+s"(k.tolA), "+v"(k.mu_nm1));
    if (LIN && SPI) __asm__ volatile("" : "+s"(k.l2c), "+v"(k.l2o), "+s"(k.l2t));
    const uint32_t hist_l = lds_addr(s.hist) + 4u * (uint32_t)((lane % k.copies) * k.nbins);
    WaveCtx c;
    c.rcount = 0;
    c.nrechk = 0;
    unsigned long long ncand = 0;
    const float far = 1.0e18f;
    // matrix-instruction lane layout: operands hold point lane % 16, component
    // lane / 16; result register i holds A point 4 (lane / 16) + i, B point lane % 16
    const int lcol = lane & 15, lk = lane >> 4;
    const uint32_t lane_id = ((uint32_t)lcol << 6) | ((uint32_t)lk << 2);

    unsigned long long wave_pairs = 0;  // pairs claimed since this wave last emptied the histogram
    uint32_t wave_tested = 0;           // weighted: pairs tested since then
    unsigned long long nflush = 0;      // merges made by this wave before the end
    const unsigned long long flush_pairs = a.flush_pairs;
    uint32_t out_off = 0;               // first bin of the current catalogue in the outputs
    // u32 overflow guard of the LDS histogram: every wave empties it (atomic
    // exchange) after claiming flush_pairs <= 2^26 pairs, so it never holds
    // more than 16 (2^26 + 128 x 2^19) = 2^31 increments (items hold at most
    // 128 x b_chunk pairs, b_chunk <= 2^19).  Weighted words hold less: a wave
    // also empties them once it has tested wf.limit pairs since it last did.
    auto exchange_out = [&]() __attribute__((always_inline)) {
        nflush++;
        if (W) {
            for (int b = lane; b < k.nbins; b += 64) {
                const unsigned long long lo = lds_exch_u64(s.wl + 8u * (uint32_t)b);
                const unsigned long long hi = lds_exch_u64(s.wl + 8u * (uint32_t)b + s.wstride);
                if (!(lo | hi)) continue;
                __int128 v;
                const uint32_t n = weight_words(k.wf, lo, hi, v);
                if (n) atomicAdd(&a.out_counts[out_off + b], (unsigned long long)n);
                add_out_w(&a.out_w[2 * ((size_t)out_off + b)], v);
            }
            return;
        }
        for (int b = lane; b < k.nbins * k.copies; b += 64) {
            uint32_t v = atomicExch(&s.hist[b], 0u);
            if (v) atomicAdd(&a.out_counts[out_off + b % k.nbins], (unsigned long long)v);
        }
    };
    // workgroup-wide merge of the LDS histograms into the outputs, then clear
    auto merge_out = [&]() __attribute__((always_inline)) {
        for (int b = tid; b < k.nbins; b += nthr) {
            if (W) {
                const unsigned long long lo = lds_exch_u64(s.wl + 8u * (uint32_t)b);
                const unsigned long long hi = lds_exch_u64(s.wl + 8u * (uint32_t)b + s.wstride);
                if (!(lo | hi)) continue;
                __int128 v;
                const uint32_t n = weight_words(k.wf, lo, hi, v);
                if (n) atomicAdd(&a.out_counts[out_off + b], (unsigned long long)n);
                add_out_w(&a.out_w[2 * ((size_t)out_off + b)], v);
                continue;
            }
            uint32_t cnt = 0;
            for (int r = 0; r < k.copies; r++) {
                cnt += s.hist[r * k.nbins + b];
                s.hist[r * k.nbins + b] = 0u;
            }
            if (cnt) atomicAdd(&a.out_counts[out_off + b], (unsigned long long)cnt);
        }
    };
    auto drain_rechecks = [&]() __attribute__((always_inline)) {
        while (c.rcount > 0) {
            const int n = c.rcount < 64 ? c.rcount : 64;
            wave_sync_lds();
            process_rechecks<KIND, LOS, W>(a, s, c.rcount - n, n, lane, c.nrechk);
            wave_sync_lds();
            c.rcount -= n;
        }
    };
    // The pairs of the A points a0 .. a0 + cnt - 1 (one per lane) with the
    // item's B points.
    //
    // What bounds it: vector instruction issue.  Testing every candidate on the
    // vector ALU took 12.5 instructions per 64 candidates (three subtractions, a
    // product, two fmas, the compare, and the compaction), and only one candidate
    // in 3 to 10 is in range.  Here
    //  1. B points are dropped, 64 at a time and one per lane, when they lie
    //     beyond reach of the box around the A points (a quarter to a half of
    //     them: the work list only cuts whole rows and their ends);
    //  2. the others are staged in LDS, and groups of 16 meet the 64 A points
    //     on the matrix cores: one v_mfma_f32_16x16x4_f32 gives 256 squared
    //     separations |a|^2 - 2 a.b + |b|^2 in a frame centred on the A points
    //     (FP32 throughout).  The vector ALU only compares and compacts;
    //  3. the threshold has a margin above the error of that form, so every
    //     pair in range passes, and bin_queue forms the pair itself.
    // Per 64 counted pairs of an unweighted (s, mu) mock that took 68 instructions
    // before and 54 now; with the LDS claims below, on MI355X (kernel times):
    // mock of 200,003 points 1.76 -> 1.14 ms, 10M points in 50 log bins 3.97 ->
    // 2.95 ms, 1M weighted points 6.36 -> 5.01 ms, 200k x 4M weighted survey (mid
    // point) 119 -> 80 ms, tree survey 7.65 -> 4.49 ms.
    // All of this works in units of a power of two near the reach (CountArgs.f_sig),
    // so that no square or sentinel leaves FP32 whatever unit the coordinates have.
    // (s_perp, pi) counts also bound the second axis: dz for the z line of
    // sight; for the mid-point one, the difference of the two distances
    // dr = |b| - |a| from the observer.  With
    // T = d^2 - dr^2:  |a + b|^2 = (|a| + |b|)^2 - T, so pi^2 = dr^2 / (1 - T /
    // (|a| + |b|)^2) >= dr^2 and s_perp^2 = T (1 - eta), eta = dr^2 / ((|a| +
    // |b|)^2 - T), bounded over the pairs of the A points.
    auto process_half = [&](const Item& item, uint32_t a0, uint32_t cnt) __attribute__((always_inline)) {
        const int idy = (int)(int8_t)(item.meta & 0xffu);
        const int idz = (int)(int8_t)((item.meta >> 8) & 0xffu);
        const int sxi = (int)((item.meta >> 16) & 3u) - 1;
        const bool samerow = AUTO && ((item.meta >> 24) & ITEM_SAMEROW);
        const uint32_t b_begin = item.b_begin;
        const uint32_t b_end = item.b_end;
        // same-row items count b > a: nothing before a0 can pair
        uint32_t jc = samerow ? max(b_begin, a0) : b_begin;
        if (jc >= b_end) return;
        const bool av_ok = (uint32_t)lane < cnt;
        const float4 av = a.posA[a0 + (av_ok ? (uint32_t)lane : 0u)];
        float4 aabs = make_float4(0.f, 0.f, 0.f, 0.f);
        if (MID) aabs = a.absA[a0 + (av_ok ? (uint32_t)lane : 0u)];
        // B points arrive 64 at a time, one per lane, by buffer loads issued a
        // whole batch ahead.  The buffer covers the item's B range; offsets
        // past it read zeros.
        const __amdgpu_buffer_rsrc_t rB = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(a.posB + b_begin), (short)0, (int)((b_end - b_begin) * 16u), BUFFER_RSRC_WORD3);
        const uint32_t lane16 = (uint32_t)lane * 16u;
        float4 bnext = load_b(rB, lane16, (jc - b_begin) * 16u);
        double wnext = 0.0;
        if (W) {
            wnext = a.wB[min(jc + (uint32_t)lane, b_end - 1u)];
            s.swa[lane] = a.wA[a0 + (av_ok ? (uint32_t)lane : 0u)];
        }
        const float Dy = (float)idy * k.side32;
        const float Dz = (float)idz * k.side32;
        int4 ja = make_int4(0, 0, 0, 0);
        int cref = 0;
        float fx = av.x;
        if (TREE) {
            ja = ldc_i4(a.leaf_orgA, item.tile);
        } else {
            const int acx = __float_as_int(av.w);
            cref = __builtin_amdgcn_readfirstlane(acx);
            fx = av.x + (float)(acx - cref) * k.side32;
        }
        // Box around the A points: in a grid the row's cell in y and z, and in x the
        // first and last point (sorted by x to a.xstep); in a tree the points
        // themselves (lanes past the last repeat the first point).
        float x0, x1, y0 = 0.f, y1 = k.side32, z0 = 0.f, z1 = k.side32;
        if (TREE) {
            x0 = wave_min_f(fx);
            x1 = wave_max_f(fx);
            y0 = wave_min_f(av.y);
            y1 = wave_max_f(av.y);
            z0 = wave_min_f(av.z);
            z1 = wave_max_f(av.z);
        } else {
            x0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(fx), 0)) - a.xstep;
            x1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(fx), (int)cnt - 1)) + a.xstep;
        }
        const float cx = uniform_f(0.5f * (x0 + x1)), hx = uniform_f(x1 - cx);
        const float cy = uniform_f(0.5f * (y0 + y1)), hy = uniform_f(y1 - cy);
        const float cz = uniform_f(0.5f * (z0 + z1)), hz = uniform_f(z1 - cz);
        // thresholds with the margin of the frame's FP32 errors: the squared
        // separation of points within W = 2 |half box| + reach of each other, and
        // for trees the rounding of coordinates up to f_ext from their leaf's origin
        const float wsum = 2.0f * (hx + hy + hz) + 4.0f * k.side32 + a.f_reach;
        const float wext = TREE ? wsum + a.f_ext : wsum;
        const float sig = a.f_sig;  // (from here on thresholds are in the filter's unit)
        const float slack = a.f_slack * (sig * wsum) * (sig * wext);
        float t2 = a.f_t2 + slack;  // squared separation (transverse part for (s_perp, pi))
        const float c2 = a.f_cull2 + slack;
        const float cull2 = uniform_f(c2 * a.f_inv2);
        float ulim = a.f_u + a.f_uslack * (sig * wext);
        const float ucull = uniform_f(ulim * a.f_inv);
        if (LIN) {
            // Positions in the frame of the tile's first cell: over S = (x1 - x0) /
            // side + 1 cells the roundings of one displacement component come to
            // u ((10 + 6 S) side + 4 r), against the e the tolerances were derived with
            float widen = 1.0f;
            if (!TREE) {
                const float eh = (16.0f * k.side32 + 6.0f * (x1 - x0) + 4.1f * a.f_reach) * a.e_unit;
                widen = fmaxf(1.0f, eh);
            }
            c.t1 = uniform_f(k.l1t * widen);
            if (KIND == FCFC_BIN_S_MU) {
                c.tA = uniform_f(k.tolA * widen);
                c.tC = k.tolC_v * widen;
            }
            if (SPI) {
                c.t2 = uniform_f(k.l2t * widen);
                if (MID) c.t1a = k.l1a * widen;
            }
        }
        const float X = av_ok ? sig * (fx - cx) : far, Y = av_ok ? sig * (av.y - cy) : far,
                    Z = av_ok ? sig * (av.z - cz) : far;
        // second coordinate u: z, or the distance from the observer
        float Fx = 0.f, Fy = 0.f, Fz = 0.f, ua = 0.f, ulo = 0.f, uhi = 0.f, uon = 1.f;
        if (SPI && MID) {
            Fx = uniform_f(sig * (aabs.x - (fx - cx)));  // the frame's origin as seen by the observer
            Fy = uniform_f(sig * (aabs.y - (av.y - cy)));
            Fz = uniform_f(sig * (aabs.z - (av.z - cz)));
            const float ax = sig * aabs.x, ay = sig * aabs.y, az = sig * aabs.z;
            ua = __builtin_amdgcn_sqrtf(__builtin_fmaf(az, az, __builtin_fmaf(ay, ay, ax * ax)));
            // |a| + |b| of a pair in range is at least smin; where it does not exceed
            // the reach twice over, the sphere alone filters (u = 0 for every point)
            const float umin = wave_min_f(ua), umax = wave_max_f(ua);
            const float smin = 2.0f * umin - ulim, s2 = smin * smin;
            if (smin > 0.f && s2 >= 4.0f * a.f_cull2) {
                const float eta = 1.0001f * a.f_u * a.f_u / (s2 - a.f_cull2);
                t2 = a.f_t2 / (1.0f - eta) + a.f_ts + slack;
                ulim += a.f_uerr;
            } else {
                uon = 0.f;
                t2 = c2;
                ulim = 1.0f;
            }
            ulo = uon * umin - ulim;
            uhi = uon * umax + ulim;
            ua *= uon;
        }
        t2 = uniform_f(t2);
        ulim = uniform_f(ulim);
        // operands: A point lane % 16 of each group of 16, component lane / 16
        f32x4 aop, uop = {0.f, 0.f, 0.f, 0.f};
        {
            const float aa = (SPI && !MID) ? __builtin_fmaf(Y, Y, X * X)
                                           : __builtin_fmaf(Z, Z, __builtin_fmaf(Y, Y, X * X));
            s.sa[lane] = make_float4(-2.0f * X, -2.0f * Y, (SPI && !MID) ? 0.f : -2.0f * Z, aa);
            wave_sync_lds();
#pragma unroll
            for (int m = 0; m < 4; m++) aop[m] = ((const float*)s.sa)[4 * (16 * m + lcol) + lk];
            if (SPI) {
                wave_sync_lds();
                ((float*)s.sa)[lane] = MID ? ua : Z;
                wave_sync_lds();
#pragma unroll
                for (int m = 0; m < 4; m++) {
                    const float u = ((const float*)s.sa)[16 * m + lcol];
                    uop[m] = lk == 3 ? -u : (lk == 2 ? 1.0f : 0.0f);
                }
            }
            wave_sync_lds();
            const float dcell = TREE ? 0.f : (float)(__float_as_int(av.w) - cref + 64);
            s.sa[lane] = TREE ? av : make_float4(LIN ? fx : av.x, av.y - Dy, av.z - Dz, dcell);
            if (MID) s.sabs[lane] = make_float4(2.0f * aabs.x, 2.0f * aabs.y, 2.0f * aabs.z, 0.f);
        }
        // this lane's component of a staged B point in the A frame: the stored
        // component, plus the cell for x, plus an offset
        const float selside = (!TREE && !LIN && lk == 0) ? k.side32 : 0.f;
        const float off_k = sig * (lk == 0 ? -cx : (lk == 1 ? (TREE ? 0.f : Dy) - cy : (TREE ? 0.f : Dz) - cz));
        const float F_k = lk == 0 ? Fx : (lk == 1 ? Fy : Fz);
        float sigv = sig;
        if (W) __asm__ volatile("" : "+v"(sigv));  // (weighted counts have vector registers to spare)
        int ns = 0;  // staged B points waiting
        for (;;) {
            // ---- cull and stage the next 64 B points ----
            const float4 b = bnext;
            const uint32_t j = jc + (uint32_t)lane;
            const bool more = jc + 64u < b_end;
            const double wj = wnext;
            if (more) {
                bnext = load_b(rB, lane16, (jc + 64u - b_begin) * 16u);
                if (W) wnext = a.wB[min(jc + 64u + (uint32_t)lane, b_end - 1u)];
            }
            float bx, by, bz;  // in the frame centred on the A points
            float sx = b.x, sy = b.y, sz = b.z;  // as staged
            uint32_t bw = (j - b_begin) << 11;
            if (TREE) {
                const uint32_t leaf = min(j / a.tree_leaf, a.tree_nleafB - 1u);
                const int4 jb = a.leaf_orgB[leaf];
                sx = b.x + (float)(jb.x - ja.x) * a.tree_q;
                sy = b.y + (float)(jb.y - ja.y) * a.tree_q;
                sz = b.z + (float)(jb.z - ja.z) * a.tree_q;
                bx = sx - cx;
                by = sy - cy;
                bz = sz - cz;
            } else {
                const int dc = __float_as_int(b.w) + sxi * k.nx - cref;
                const float fx1 = b.x + (float)dc * k.side32;
                bx = fx1 - cx;
                by = b.y + (Dy - cy);
                bz = b.z + (Dz - cz);
                if (LIN) sx = fx1;
                else bw |= (uint32_t)((dc + 64) & 255);
            }
            const float ux = fmaxf(fabsf(bx) - hx, 0.f), uy = fmaxf(fabsf(by) - hy, 0.f),
                        uz = fmaxf(fabsf(bz) - hz, 0.f);
            bool keep = j < b_end;
            if (SPI && !MID) {
                keep = keep & (__builtin_fmaf(uy, uy, ux * ux) < cull2) & (uz < ucull);
            } else {
                keep = keep & (__builtin_fmaf(uz, uz, __builtin_fmaf(uy, uy, ux * ux)) < cull2);
            }
            if (SPI && MID) {
                const float px = __builtin_fmaf(bx, sig, Fx), py = __builtin_fmaf(by, sig, Fy),
                            pz = __builtin_fmaf(bz, sig, Fz);
                const float ub = uon * __builtin_amdgcn_sqrtf(
                                           __builtin_fmaf(pz, pz, __builtin_fmaf(py, py, px * px)));
                keep = keep & (ub > ulo) & (ub < uhi);
            }
            const uint64_t km = __builtin_amdgcn_ballot_w64(keep);
            if (keep) {
                const int slot = ns + (int)lane_prefix(km);
                s.sb[slot] = make_float4(sx, sy, sz, __uint_as_float(bw));
                if (W) s.swb[slot] = wj;
            }
            const int added = (int)__popcll(km);
            ns += added;
            ncand += (unsigned long long)((uint32_t)added * cnt);
            if (W) {
                wave_tested += (uint32_t)added * cnt;
                if (wave_tested >= k.wf.limit) {
                    wave_tested = (uint32_t)added * cnt;
                    exchange_out();
                }
            }
            jc += 64u;
            wave_sync_lds();
            // ---- whole groups of 16 staged points (the rest too at the end) ----
            // A step is 16 B points against 16 A points, one matrix instruction and
            // 256 candidates; the queue is emptied in between while it holds 64 pairs.
            const int ng = more ? (ns >> 4) : ((ns + 15) >> 4);
            uint32_t qend = s.qbase;  // LDS byte address of the queue's end
            const uint32_t qfull = s.qbase + 128u;
            const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
            auto empty = [&](uint32_t down_to) __attribute__((always_inline)) {
                while (qend > down_to) {
                    const int n = min((int)(qend - s.qbase) >> 1, 64);
                    qend -= 2u * (uint32_t)n;
                    wave_sync_lds();
                    bin_queue<KIND, LOS, W, TREE, LIN>(a, k, s, hist_l, qend, n, lane, c);
                    wave_sync_lds();
                }
            };
            for (int g = 0; g < ng; g++) {
                // the operands of the next 16 B points
                const int slot = 16 * g + lcol;
                const uint32_t sat = s.wbase + OFF_SB + 16u * (uint32_t)slot;
                float v = lds_f1(sat + 4u * (uint32_t)lk);
                const uint32_t w = __float_as_uint(lds_f1(sat + 12u));
                if (!TREE && !LIN) v = __builtin_fmaf((float)(w & 255u) - 64.0f, selside, v);
                v = __builtin_fmaf(v, sigv, off_k);
                // slots past the last staged point (stale memory) become the origin with
                // a |b|^2 out of every reach
                const bool staged = slot < ns;
                v = staged ? v : 0.f;
                const float bop = lk == 3 ? 1.0f : v;
                // |b|^2 of point lane % 16 in every lane: a product with ones
                float sq = lk < ((SPI && !MID) ? 2 : 3) ? v * v : 0.f;
                sq = staged ? sq : 1.0e37f;
                const f32x4 bb = __builtin_amdgcn_mfma_f32_16x16x4f32(1.0f, sq, zero, 0, 0, 0);
                float bu = bop;  // u = z: component 2, and the one of component 3
                if (SPI && MID) {
                    const float pc = lk == 3 ? 0.f : v + F_k;
                    const f32x4 rr = __builtin_amdgcn_mfma_f32_16x16x4f32(1.0f, pc * pc, zero, 0, 0, 0);
                    bu = lk == 2 ? uon * __builtin_amdgcn_sqrtf(rr[0]) : (lk == 3 ? 1.0f : 0.f);
                }
                // same-row items count b > a: the B point's rank against the A slots
                const int rel = AUTO ? (int)(b_begin + (w >> 11) - a0) - 4 * lk : 0;
                const uint32_t gid = lane_id + ((uint32_t)g << 10);
#pragma unroll
                for (int m = 0; m < 4; m++) {
                    f32x4 d = __builtin_amdgcn_mfma_f32_16x16x4f32(aop[m], bop, bb, 0, 0, 0);
                    f32x4 du = zero;
                    if (SPI) du = __builtin_amdgcn_mfma_f32_16x16x4f32(uop[m], bu, zero, 0, 0, 0);
                    if (AUTO && samerow) {
#pragma unroll
                        for (int i = 0; i < 4; i++) d[i] = rel > 16 * m + i ? d[i] : 1.0e37f;
                    }
                    // result register i: A slot 16 m + 4 (lane / 16) + i, B slot lane % 16 of the group
#pragma unroll
                    for (int i = 0; i < 4; i++) {
                        float t = d[i];
                        if (SPI && MID) t = __builtin_fmaf(-du[i], du[i], t);
                        uint64_t in = __builtin_amdgcn_ballot_w64(t < t2);
                        if (SPI) in &= __builtin_amdgcn_ballot_w64(fabsf(du[i]) < ulim);
                        queue_append(qend, in, gid + (uint32_t)(16 * m + i));
                    }
                    // the queue holds 63 pairs and those of one matrix instruction; what is
                    // left of it at the end of the staged points is emptied with the last
                    if (qend >= qfull || (m == 3 && g + 1 == ng)) empty(m == 3 && g + 1 == ng ? s.qbase : qfull - 2u);
                }
            }
            if (!more) break;
            // the staged points past the last whole group go to the front
            const int done = ng * 16;
            const int left = ns - done;
            if (done > 0 && left > 0) {
                float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
                double tw = 0.0;
                if (lane < left) {
                    t = s.sb[done + lane];
                    if (W) tw = s.swb[done + lane];
                }
                wave_sync_lds();
                if (lane < left) {
                    s.sb[lane] = t;
                    if (W) s.swb[lane] = tw;
                }
                wave_sync_lds();
            }
            ns = left;
        }
        wave_sync_lds();
    };
    // Process items handed out by grab() (an index, or ~0u when there are no
    // more), claimed two ahead.
    auto process_items = [&](auto grab) __attribute__((always_inline)) {
    uint32_t cur_it = grab();
    // timing: an item's time runs from its start to the next item's start on
    // this wave (fetch and loop overhead included), the last one to the end
    unsigned long long t_prev = 0;
    uint32_t prev_it = ~0u;
    while (cur_it != ~0u) {
        const uint32_t it = cur_it;
        if (a.times && lane == 0) {
            const unsigned long long t = wall_clock64();
            if (prev_it != ~0u) a.times[prev_it] = (uint32_t)min<unsigned long long>(t - t_prev, 0xffffffffull);
            t_prev = t;
            prev_it = it;
        }
        const uint32_t nxt_it = grab();
        const Item cur = ldc_item(a.items, it);
        const uint32_t acnt = cur.a_count;
        c.it = it;
        wave_pairs += (uint64_t)acnt * (uint64_t)(cur.b_end - cur.b_begin);
        if (wave_pairs >= flush_pairs) {
            wave_pairs = 0;
            wave_tested = 0;
            exchange_out();
        }
        for (uint32_t h = 0; h < acnt; h += 64u) {
            c.aslot0 = h;
            process_half(cur, cur.a_begin + h, min(acnt - h, 64u));
        }
        cur_it = nxt_it;
    }
    if (a.times && lane == 0 && prev_it != ~0u)
        a.times[prev_it] = (uint32_t)min<unsigned long long>(wall_clock64() - t_prev, 0xffffffffull);
    };
    if (!BATCH) {
        const uint32_t nitems = __builtin_amdgcn_readfirstlane(*a.nitems_dev);
        const uint32_t sc = a.shard_count, si = a.shard_index;
        // Every wave of the device claiming work on one cursor is a bound of its own
        // for lists of short items: the atomics serialise at about 12 ns each on
        // MI355X (5.2 ms for the 437,000 items of 10M points in 50 log bins, which
        // count in 3.2 ms).  So a workgroup claims up to 16 consecutive positions at
        // a time (neighbouring tiles and rows; fewer towards the end of the list, so
        // that all workgroups finish together) and its waves take them from LDS.
        // Dealing the list out in advance instead left workgroups up to 20 % apart:
        // items of one cost differ several-fold in the pairs they count.
        const uint32_t npos = nitems > si ? (nitems - si + sc - 1u) / sc : 0u;  // this shard's positions
        WorkClaim wc(s.misc);
        process_items([&]() -> uint32_t {
            uint32_t pos = ~0u;
            if (lane == 0) {
                while (!wc.take(pos) && !wc.drained()) {
                    if (!wc.lock()) {
                        __builtin_amdgcn_s_sleep(1);
                        continue;
                    }
                    if (wc.empty()) {
                        const uint32_t seen = wc.end();  // 0 at first
                        const uint32_t rest = seen < npos ? npos - seen : 0u;
                        const uint32_t want = min(16u, max(1u, rest / ((seen ? 2u : 1u) * gridDim.x)));
                        const uint32_t at = atomicAdd(a.cursor, want);
                        wc.refill(at, min(at + want, npos), npos);
                    }
                    wc.unlock();
                }
            }
            pos = __builtin_amdgcn_readfirstlane(pos);
            return pos == ~0u ? ~0u : pos * sc + si;
        });
        drain_rechecks();
        __syncthreads();
        merge_out();
    } else {
        // Workgroup-synchronous chunks of items of one catalogue at a time: the
        // LDS histograms always belong to the workgroup's current catalogue.
        uint32_t* sm32 = (uint32_t*)(s.misc + 1);  // [0] chunk, [1] cursor within the chunk
        const uint32_t nchunks = __builtin_amdgcn_readfirstlane(*a.nchunks_dev);
        uint32_t cur_cat = ~0u;
        for (;;) {
            if (tid == 0) {
                sm32[0] = atomicAdd(a.chunk_cursor, 1u);
                sm32[1] = 0u;
            }
            __syncthreads();
            const uint32_t chunk = __builtin_amdgcn_readfirstlane(sm32[0]);
            if (chunk >= nchunks) break;
            // chunk -> position in the catalogue order (binary search on the chunk prefix)
            int lo = 0, hi = a.ncat;
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (ldc_u32(a.chunk_prefix, (uint32_t)mid) <= chunk) lo = mid;
                else hi = mid;
            }
            const uint32_t cat = ldc_u32(a.cat_order, (uint32_t)lo);
            const uint32_t local = chunk - ldc_u32(a.chunk_prefix, (uint32_t)lo);
            const uint32_t ib = ldc_u32(a.cat_items, cat) + local * (uint32_t)a.chunk_items;
            const uint32_t ie_cat = ldc_u32(a.cat_items, cat + 1u);
            const uint32_t ie = min(ib + (uint32_t)a.chunk_items, ie_cat);
            if (cat != cur_cat) {
                if (cur_cat != ~0u) merge_out();
                __syncthreads();
                cur_cat = cat;
                out_off = cat * (uint32_t)k.nbins;
            }
            process_items([&]() -> uint32_t {
                uint32_t v = 0;
                if (lane == 0) v = atomicAdd(&sm32[1], 1u);
                v = __builtin_amdgcn_readfirstlane(v) + ib;
                return v < ie ? v : ~0u;
            });
            drain_rechecks();
            __syncthreads();
        }
        if (cur_cat != ~0u) merge_out();
    }
    if (lane == 0 && a.stats) {
        atomicAdd(&a.stats[0], ncand);
        atomicAdd(&a.stats[1], c.nrechk);
        if (nflush) atomicAdd(&a.stats[6], nflush);
    }
}

typedef void (*CountKernel)(const CountArgs*);

// The instantiations with computed bins (uniform edges on every axis) and with
// look-up tables, each built in a source file of its own.  Batched counts use
// the auto instantiation for cross pairs too, since only items of an auto
// pair carry the same-row flag.
CountKernel count_kernel_lin(int mode, int kind, int los, bool is_auto, bool w);
CountKernel count_kernel_lut(int mode, int kind, int los, bool is_auto, bool w);

template <int KIND, int LOS, int MODE, bool LIN>
static CountKernel count_kernel_aw(bool is_auto, bool w) {
    if constexpr (MODE != COUNT_BATCH) {
        if (!is_auto) return w ? k_count<KIND, LOS, false, true, MODE, LIN> : k_count<KIND, LOS, false, false, MODE, LIN>;
    }
    return w ? k_count<KIND, LOS, true, true, MODE, LIN> : k_count<KIND, LOS, true, false, MODE, LIN>;
}
template <int KIND, int LOS, bool LIN>
static CountKernel count_kernel_mode(int mode, bool is_auto, bool w) {
    if (mode == COUNT_TREE) return count_kernel_aw<KIND, LOS, COUNT_TREE, LIN>(is_auto, w);
    if (mode == COUNT_BATCH) return count_kernel_aw<KIND, LOS, COUNT_BATCH, LIN>(is_auto, w);
    return count_kernel_aw<KIND, LOS, COUNT_SINGLE, LIN>(is_auto, w);
}
template <bool LIN>
static CountKernel count_kernel_pick(int mode, int kind, int los, bool is_auto, bool w) {
    const bool mid = los == FCFC_LOS_MIDPOINT;
    if (kind == FCFC_BIN_S) return count_kernel_mode<FCFC_BIN_S, FCFC_LOS_Z, LIN>(mode, is_auto, w);
    if (kind == FCFC_BIN_S_MU)
        return mid ? count_kernel_mode<FCFC_BIN_S_MU, FCFC_LOS_MIDPOINT, LIN>(mode, is_auto, w)
                   : count_kernel_mode<FCFC_BIN_S_MU, FCFC_LOS_Z, LIN>(mode, is_auto, w);
    return mid ? count_kernel_mode<FCFC_BIN_SPERP_PI, FCFC_LOS_MIDPOINT, LIN>(mode, is_auto, w)
               : count_kernel_mode<FCFC_BIN_SPERP_PI, FCFC_LOS_Z, LIN>(mode, is_auto, w);
}

}  // namespace fcfc
