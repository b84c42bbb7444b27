// sg_nbr.hip -- neighbour lists of the gas (the lists the paper's DC and HFC
// kernels build from CellSPH / indexPC / hmaxCell, Sec. 3), stored as CSR
// by sorted slot.
//
// Search region.  For every non-empty level l a target s must scan the
// cells within R = (h_s + hmax_l)(1 + 2^-10) of itself: any pair passing
// the predicate has |r| < (h_s + h_t)(1 + 2^-20) <= R, so the scan is
// complete.  Cells with the same (level, z, y) and consecutive x are
// consecutive in key order, so each (z, y) row of a box of cells is one
// contiguous slot range, and visiting levels, then z, y, x in ascending
// order yields candidates in ascending slot order: rows need no sort.
//
// Cell-staged search (k_nbr_search).  One wavefront takes 1 to 32 consecutive
// target slots and walks them cell by cell: the targets that share a cell
// key form a run, and the run's search region is the union (per level) of
// its targets' boxes.  The rows of that region are flattened into one
// candidate stream, loaded 192 candidates at a time (three per lane) and
// held in registers while every target of the run tests them, so a
// candidate is fetched once per cell instead of once per target.  Any
// grouping gives the same lists: the union contains each target's own box,
// and every target keeps only the candidates that pass its predicate, in
// stream order.  The union of the targets' reaches is a DPP reduction per
// dimension, its boxes on all levels are computed at once (four lanes a
// level), the stream offsets are a DPP scan of the row lengths, and the
// slots of a chunk's stream positions a running maximum over marks that the
// rows leave where they start.
//
// Bound by instruction issue: the scalar unit, which a compute unit's four
// SIMDs share, as much as the vector ALUs (1190 candidates a target for 48
// neighbours: a large part of a run's box is out of a given target's reach).
// So the loop over targets and candidates has one branch per 192 candidates
// while there is no hit, masks are combined only for batches with one, and
// candidates are tested by the FP32 pretest below.  Search at 1048576
// targets, per target: 264 scalar, 66 branch and 377 vector instructions
// before, 149, 42 and 272 now; with two more wavefronts a SIMD (64 VGPRs),
// 731 -> 490 us.  (The pretest alone, in a loop with a branch and two mask
// operations a batch, was slower than the predicate: 820 us.)
//
// Each target writes its hits into a slot of its own, kSlot entries long,
// in a scratch array (no atomics), and counts them.  A scan of the counts
// gives the CSR offsets; a copy pass then moves every slot to its CSR row,
// and a target with more than kSlot hits (none in the collision workloads:
// at most 58 at 2M particles; clustered gas can have thousands) searches a
// second time, alone, straight into its row.
//
// Built with -ffp-contract=off: the FP32 predicate must round exactly as
// specified (each product and fma rounded once).
#include <type_traits>

#include "sg_internal.h"

namespace {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / 64;
// Targets per wavefront of the search, NT (lanes 0 .. NT-1 hold them; all
// 64 lanes hold candidates): 32 at a million targets, down to 1 for a few
// thousand, by the number of targets (sg_nbr_targets below has the times).
// Candidate batches held in registers per target pass: each target's data
// is read and its hit count fetched once per kHold batches instead of once
// per batch.  Search stage at 2M particles when the target data were lane
// reads (about 23 instead of 28 vector instructions per 64 pair tests):
// 1.53 ms with one batch, 1.41 with 2, 1.32 with 4, 1.49 with 8 (113 VGPRs:
// 4 waves per SIMD).  With the set-up as it is now: 2: 0.98-0.99 ms, 3:
// 0.94 (63 VGPRs), 4: 0.96, 6: 1.01-1.02.  With the pretest, stage at
// 1048576 targets: 2: 0.775, 3: 0.741, 4: 0.728 at 6 wavefronts a SIMD, 3:
// 0.716 at 8.
constexpr int kHold = 3;
// Targets per wavefront from which the pretest is used: it pays for the
// candidates' conversion from a few targets a run on (stage at 9001 targets
// with 1 / 2: 47 / 52 us without, 51 / 51 with it; 262144, 2: 427 / 453).
constexpr int kPreMin = 4;

__device__ inline unsigned rank_below(unsigned long long mask) {
    return __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
}

// xi_ij < 2 tested in FP32: see the grid / neighbour contract in sphgrav.h.
__device__ inline bool nbr_pred(double xi, double yi, double zi, float hif, double xj, double yj,
                                double zj, double hj) {
    const float dx = (float)(xi - xj);
    const float dy = (float)(yi - yj);
    const float dz = (float)(zi - zj);
    const float dxx = dx * dx;
    const float r2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dxx));
    const float cut = hif + (float)hj;
    const float cut2 = cut * cut;
    return r2 < cut2;
}

// The same predicate with the candidate's h already rounded to FP32.
__device__ inline bool nbr_pred_f(double xi, double yi, double zi, float hif, double xj,
                                  double yj, double zj, float hjf) {
    const float dx = (float)(xi - xj);
    const float dy = (float)(yi - yj);
    const float dz = (float)(zi - zj);
    const float dxx = dx * dx;
    const float r2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dxx));
    const float cut = hif + hjf;
    const float cut2 = cut * cut;
    return r2 < cut2;
}

// Pretest of the predicate in FP32, for runs of several targets.  With
// coordinates x', y', z' from an origin O close to both particles,
//   (r^2 - (h_i + h_j)^2) / 2 = a_i + a_j - x'_i x'_j - y'_i y'_j
//                               - z'_i z'_j - h_i h_j,   a = (|x'|^2 - h^2) / 2:
// four FMAs and a comparison a pair, against three FP64 subtractions, three
// conversions and six FP32 operations for the predicate itself.  Where the
// value is within kPreTol (|x'|^2 + h^2) of zero, summed over both particles,
// the pair is undecided and the predicate decides (a few pairs in a
// thousand targets).  The tolerance covers, in units of u = 2^-24 and per
// (|x'|^2 + h^2) of either particle: rounding of the coordinates 2, the
// predicate's own roundings 5, a 2.5, the four FMAs 4: 13.5 of the 32 that
// 2^-19 gives; kPreAbs covers what underflows.  A value that is not finite
// never decides against a pair that the predicate would take: comparisons
// with NaN leave it undecided.
constexpr float kPreTol = 0x1p-19f, kPreAbs = 0x1p-118f;
struct pre_rec {                           // x', y', z', h
    float x, y, z, h;
    __device__ inline float q() const {
        return __builtin_fmaf(x, x, __builtin_fmaf(y, y, z * z));
    }
    __device__ inline float tol() const { return kPreTol * __builtin_fmaf(h, h, q()); }
    __device__ inline float a() const { return 0.5f * __builtin_fmaf(-h, h, q()); }
};

constexpr int32_t kSlot = 96;              // scratch entries per target

// Cells [lo, hi] (per dimension, clamped to the grid) of level l within
// R = (h + hmax_l)(1 + 2^-10) of p; false when the level has no such cell.
__device__ inline bool level_box(const sg_grid_dev* __restrict__ g, int l, const double p[3],
                                 double h, int32_t lo[3], int32_t hi3[3]) {
    // in cell units: the reach R inv and the position (p - o) inv (their
    // rounding differs from that of (p +- R - o) inv by far less than the
    // 2^-10 margin of R, so the box still holds every cell within reach)
    const double inv = g->invL[l];
    const double Ri = (h + g->hmaxlev[l]) * (1.0 + 0x1p-10) * inv;
    bool empty = false;
    for (int d = 0; d < 3; ++d) {
        const double c = (p[d] - g->org[l][d]) * inv;
        // clamped into [-1, 2^30] first, where the conversion is exact (a
        // NaN becomes -1: an empty box)
        const int32_t a = (int32_t)fmin(fmax(floor(c - Ri), -1.0), 0x1p30);
        const int32_t b = (int32_t)fmin(fmax(floor(c + Ri), -1.0), 0x1p30);
        const int32_t top = (int32_t)g->dim[l][d] - 1;
        if (b < 0 || a > top) empty = true;
        lo[d] = min(max(a, 0), top);
        hi3[d] = min(max(b, 0), top);
    }
    return !empty;
}

// One target's scan over its own boxes (used by the overflow path).
template <typename F>
__device__ inline void nbr_scan(const sg_grid_dev* __restrict__ g, int64_t ng, int64_t s,
                                unsigned lane, const double* __restrict__ xs,
                                const double* __restrict__ ys, const double* __restrict__ zs,
                                const double* __restrict__ hs, const int64_t* __restrict__ off,
                                F&& hit) {
    const double p[3] = {xs[s], ys[s], zs[s]};
    const double hi = hs[s];
    const float hif = (float)hi;
    const int nlev = g->nlev;
    for (int l = 0; l < nlev; ++l) {
        if (g->ncell[l] == 0) continue;
        int32_t lo[3], hi3[3];
        if (!level_box(g, l, p, hi, lo, hi3)) continue;
        const int64_t base = g->base[l], dx = g->dim[l][0], dy = g->dim[l][1];
        const int64_t ny = (int64_t)hi3[1] - lo[1] + 1;
        const int64_t nrows = ((int64_t)hi3[2] - lo[2] + 1) * ny;
        for (int64_t r0 = 0; r0 < nrows; r0 += 64) {
            // bounds of rows r0 .. r0+63, one row per lane; offsets are
            // bounded by ng: clamp so that a corrupt table can never send a
            // load outside the sorted arrays
            int64_t my0 = 0, my1 = 0;
            const int64_t r = r0 + lane;
            if (r < nrows) {
                const int64_t cz = lo[2] + r / ny, cy = lo[1] + r % ny;
                const int64_t row = base + (cz * dy + cy) * dx;
                my0 = off[row + lo[0]];
                my1 = off[row + hi3[0] + 1];
                my0 = my0 < 0 ? 0 : my0;
                my1 = my1 > ng ? ng : my1;
            }
            const int nr = (int)(nrows - r0 < 64 ? nrows - r0 : 64);
            for (int k = 0; k < nr; ++k) {
                const int64_t t0 = __shfl(my0, k, 64), t1 = __shfl(my1, k, 64);
                for (int64_t tb = t0; tb < t1; tb += 64) {
                    const int64_t t = tb + lane;
                    bool ok = false;
                    if (t < t1 && t != s) ok = nbr_pred(p[0], p[1], p[2], hif, xs[t], ys[t], zs[t], hs[t]);
                    hit(__ballot(ok), t, ok);
                }
            }
        }
    }
}

// Cross-lane reductions and scan by DPP row operations (no LDS round
// trips; every lane of the wavefront must be active).  Controls:
// quad_perm [1,0,3,2] 0xb1, [2,3,0,1] 0x4e, row_shr:n 0x110 + n,
// row_mirror 0x140, row_half_mirror 0x141, row_bcast:15 0x142 (lane 15 of
// each row into the next row), row_bcast:31 0x143 (lane 31 into rows 2, 3).
template <int kCtrl, int kRowMask = 0xf>
__device__ inline int32_t dpp(int32_t old, int32_t v) {
    return __builtin_amdgcn_update_dpp(old, v, kCtrl, kRowMask, 0xf, false);
}

// inclusive prefix sum over the 64 lanes
__device__ inline int32_t wave_incl_sum(int32_t v) {
    v += dpp<0x111>(0, v);                     // within each row of 16
    v += dpp<0x112>(0, v);
    v += dpp<0x114>(0, v);
    v += dpp<0x118>(0, v);
    v += dpp<0x142, 0xa>(0, v);                // rows 1, 3: + total of rows 0, 2
    v += dpp<0x143, 0xc>(0, v);                // rows 2, 3: + total of rows 0, 1
    return v;
}

// inclusive prefix maximum over the 64 lanes, of values >= 0
__device__ inline int32_t wave_incl_max(int32_t v) {
    v = max(v, dpp<0x111>(0, v));
    v = max(v, dpp<0x112>(0, v));
    v = max(v, dpp<0x114>(0, v));
    v = max(v, dpp<0x118>(0, v));
    v = max(v, dpp<0x142, 0xa>(0, v));
    v = max(v, dpp<0x143, 0xc>(0, v));
    return v;
}

// a[i] with a 32-bit byte offset (one address register: slots of 2^29
// targets, 206 GB of scratch and as much again beside, are out of reach)
__device__ inline double at32(const double* __restrict__ a, uint32_t i) {
    return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(a) + (size_t)(i * 8u));
}

// minimum over each half of the wavefront, in its last lane (31, 63)
__device__ inline double half_min(double v) {
    auto step = [&](auto ctrl, auto rows) {
        constexpr int kCtrl = decltype(ctrl)::value, kRows = decltype(rows)::value;
        const unsigned long long q = __builtin_bit_cast(unsigned long long, v);
        const int32_t lo = dpp<kCtrl, kRows>((int32_t)(unsigned)q, (int32_t)(unsigned)q);
        const int32_t hi = dpp<kCtrl, kRows>((int32_t)(q >> 32), (int32_t)(q >> 32));
        v = fmin(v, __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
    };
    step(std::integral_constant<int, 0xb1>{}, std::integral_constant<int, 0xf>{});
    step(std::integral_constant<int, 0x4e>{}, std::integral_constant<int, 0xf>{});
    step(std::integral_constant<int, 0x141>{}, std::integral_constant<int, 0xf>{});
    step(std::integral_constant<int, 0x140>{}, std::integral_constant<int, 0xf>{});   // rows of 16
    step(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});   // rows 1, 3
    return v;
}

// v of lane l (uniform)
__device__ inline double lane_value(double v, int l) {
    const unsigned long long q = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)q, l);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(q >> 32), l);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// The search of wavefront w (target slots NT w onward); w is uniform.
template <int NT>
__device__ __attribute__((always_inline)) inline void nbr_search_wave(
    const sg_grid_dev* __restrict__ g, int64_t ng, const double* __restrict__ xs,
    const double* __restrict__ ys, const double* __restrict__ zs, const double* __restrict__ hs,
    const int64_t* __restrict__ off, const int32_t* __restrict__ perm,
    const int32_t* __restrict__ key, int32_t* __restrict__ cnt, int32_t* __restrict__ slots,
    int32_t w) {
    if (g->err & SGE_SORT_FATAL) return;
    const unsigned lane = threadIdx.x & 63;
    const int64_t g0 = (int64_t)w * NT;
    if (g0 >= ng) return;
    // target g0 + (lane & 31) in both halves of the wavefront (the upper one
    // only helps with the run's reach)
    static_assert(NT <= 32, "a target a lane, twice");
    const unsigned tl = lane & 31;
    const int64_t s = g0 + tl;
    const bool live = lane < (unsigned)NT && s < ng;
    double p[3] = {0.0, 0.0, 0.0}, h = 0.0;
    int32_t k = -1;
    if (tl < (unsigned)NT && s < ng) {
        p[0] = xs[s];
        p[1] = ys[s];
        p[2] = zs[s];
        h = hs[s];
        const int32_t i = perm[s];
        // the key only groups targets (any grouping is correct)
        k = (uint32_t)i < (uint64_t)ng ? key[i] : -2 - (int32_t)lane;
    }
    const float hif = (float)h;
    // the wavefront's targets in LDS: a target pass reads its target's
    // record with broadcast loads (one address instruction) instead of
    // seven lane reads on the vector ALU (search stage at 1M gas 1.147 ->
    // 1.096 ms); 3-4 KB per workgroup, which still fits beside the gravity
    // kernel's workgroups on a compute unit
    constexpr bool kPre = NT >= kPreMin;
    struct target_rec { double x, y, z; float h, pad; };
    struct pre_cut { float maybe, sure; };
    __shared__ target_rec tp[kPre ? 1 : kWaves][kPre ? 1 : NT];
    __shared__ pre_rec tq[kPre ? kWaves : 1][kPre ? NT : 1];
    __shared__ pre_cut tc[kPre ? kWaves : 1][kPre ? NT : 1];
    target_rec* const mytp = tp[kPre ? 0 : threadIdx.x >> 6];
    pre_rec* const mytq = tq[kPre ? threadIdx.x >> 6 : 0];
    pre_cut* const mytc = tc[kPre ? threadIdx.x >> 6 : 0];
    __shared__ int32_t mark[kWaves][64 * kHold];
    int32_t* const mymark = mark[threadIdx.x >> 6];
    if (!kPre && lane < (unsigned)NT) mytp[lane] = target_rec{p[0], p[1], p[2], hif, 0.0f};
    wave_sync();
    // end of target g0 + lane's hits, from the wavefront's first slot
    int32_t* const wslots = slots + g0 * kSlot;
    int32_t mine = (int32_t)lane * kSlot;
    const int nlev = g->nlev;
    unsigned long long todo = __ballot(live);
    while (todo) {
        const int lead = __builtin_ctzll(todo);
        const int32_t rk = __builtin_amdgcn_readlane(k, lead);
        // the slots are in key order: a run is lanes lead .. lead + nrun - 1
        const unsigned long long eq = __ballot(live && k == rk) >> lead;
        const int nrun = __builtin_ctzll(~eq);             // (NT < 64: ~eq is not 0)
        todo &= todo >> lead >> nrun << lead << nrun;
        const bool inrun = tl - (unsigned)lead < (unsigned)nrun;
        // the run's reach per dimension, from its first target O: lower end
        // min (p - O - h (1 + 2^-10)) in lane 31, minus the upper end in 63
        double O[3], rlo[3], rhi[3];
        for (int d = 0; d < 3; ++d) {
            O[d] = lane_value(p[d], lead);
            const double q = p[d] - O[d];
            double v = inrun ? (lane < 32 ? q : -q) - h * (1.0 + 0x1p-10) : __builtin_inf();
            v = half_min(v);
            rlo[d] = lane_value(v, 31);
            rhi[d] = -lane_value(v, 63);
        }
        if constexpr (kPre) {
            // pretest: coordinates from O
            if (inrun && lane < 32) {
                const pre_rec t{(float)(p[0] - O[0]), (float)(p[1] - O[1]), (float)(p[2] - O[2]), hif};
                const float m = t.tol() + kPreAbs;
                mytq[lane] = t;
                mytc[lane] = pre_cut{m - t.a(), -m - t.a()};
            }
            wave_sync();
        }
        // the boxes of cells within reach: lane 4 l + d computes dimension d
        // of level l (the run's box is the union of its targets' boxes, as
        // its reach is of theirs)
        static_assert(SG_MAXLEV <= 16, "four lanes a level");
        int32_t blo = 0, bhi = 0, bdim = 0;
        const int lv = (int)(lane >> 2), ld = (int)(lane & 3);
        bool ok = ld < 3 && lv < nlev && g->ncell[lv < SG_MAXLEV ? lv : 0] != 0;
        if (ok) {
            const double inv = g->invL[lv], hl = g->hmaxlev[lv] * (1.0 + 0x1p-10);
            const double o = (ld == 0 ? O[0] : (ld == 1 ? O[1] : O[2])) - g->org[lv][ld];
            const double a = (ld == 0 ? rlo[0] : (ld == 1 ? rlo[1] : rlo[2])) - hl;
            const double b = (ld == 0 ? rhi[0] : (ld == 1 ? rhi[1] : rhi[2])) + hl;
            bdim = (int32_t)g->dim[lv][ld];
            // clamped into [-1, 2^30] first, where the conversion is exact
            // (a NaN becomes -1: an empty box)
            const int32_t ca = (int32_t)fmin(fmax(floor((o + a) * inv), -1.0), 0x1p30);
            const int32_t cb = (int32_t)fmin(fmax(floor((o + b) * inv), -1.0), 0x1p30);
            ok = cb >= 0 && ca < bdim && ca <= cb;
            blo = max(ca, 0);
            bhi = min(cb, bdim - 1);
        }
        unsigned long long lm = __ballot(ok);
        lm &= (lm >> 1) & (lm >> 2) & 0x1111111111111111ull;
        for (; lm; lm &= lm - 1) {
            // wave-uniform, held in scalar registers so that every loop
            // below is uniform and its cross-lane reads see all lanes
            const int lb = __builtin_ctzll(lm);
            int32_t ulo[3], uhi[3];
            for (int d = 0; d < 3; ++d) {
                ulo[d] = __builtin_amdgcn_readlane(blo, lb + d);
                uhi[d] = __builtin_amdgcn_readlane(bhi, lb + d);
            }
            const int32_t dx = __builtin_amdgcn_readlane(bdim, lb);
            const int32_t dy = __builtin_amdgcn_readlane(bdim, lb + 1);
            const int64_t base = g->base[lb >> 2];
            const uint32_t ny = (uint32_t)(uhi[1] - ulo[1] + 1);
            const int32_t nrows = (int32_t)((uint32_t)(uhi[2] - ulo[2] + 1) * ny);
            const float rny = __builtin_amdgcn_rcpf((float)ny);
            for (int32_t r0 = 0; r0 < nrows; r0 += 64) {
                // rows r0 .. r0+63, one per lane: first slot and length
                // (offsets clamped to [0, ng] so that a corrupt table can
                // never send a load outside the sorted arrays); row and
                // cell indices fit int32 (a level's cell count does)
                int32_t first = 0, len = 0;
                const int32_t r = r0 + (int32_t)lane;
                if (r < nrows) {
                    // (exact below 2^20: (r + 1/2) / ny is at least 1 / (2 ny)
                    // from a whole number)
                    const uint32_t rz = nrows <= 1 << 20 ? (uint32_t)(((float)r + 0.5f) * rny)
                                                         : (uint32_t)r / ny;
                    const int32_t cz = ulo[2] + (int32_t)rz, cy = ulo[1] + (int32_t)((uint32_t)r - rz * ny);
                    const int64_t row = base + (int64_t)((cz * dy + cy) * dx);
                    int64_t a = off[row + ulo[0]], b = off[row + uhi[0] + 1];
                    a = a < 0 ? 0 : (a > ng ? ng : a);
                    b = b < a ? a : (b > ng ? ng : b);
                    first = (int32_t)a;
                    len = (int32_t)(b - a);
                }
                // flatten: the rows are disjoint slot ranges, so the total
                // is at most ng
                const int32_t incl = wave_incl_sum(len);
                const int32_t start = incl - len;
                const int32_t total = __builtin_amdgcn_readlane(incl, 63);
                // a row's slots are its stream positions plus fs, which
                // never falls along the rows (they ascend)
                const int32_t fs = first - start;
                int32_t carry = 0;
                // candidates in chunks of kHold batches of 64, held in
                // registers while each target of the run tests the whole
                // chunk (its record read from LDS once per chunk, its hit
                // count carried in a scalar register)
                for (int32_t cb0 = 0; cb0 < total; cb0 += 64 * kHold) {
                    // slots of the chunk's stream positions: each non-empty
                    // row puts its fs where it starts, and a running maximum
                    // carries it over the row (against a walk over the rows
                    // with two lane reads each: the scalar unit, which four
                    // SIMDs share, was what bounded the search)
#pragma unroll
                    for (int k = 0; k < kHold; ++k) mymark[64 * k + lane] = 0;
                    if (len > 0 && start >= cb0 && start < cb0 + 64 * kHold) mymark[start - cb0] = fs;
                    wave_sync();
                    int32_t tk[kHold];
                    unsigned long long vm[kHold];          // lanes holding a candidate
                    double xd[kHold], yd[kHold], zd[kHold], hd[kHold];
                    // every batch's loads are issued before any is used
                    // (h converts to FP32 after the last one); lanes past
                    // the stream load a clamped slot and are masked out
#pragma unroll
                    for (int k = 0; k < kHold; ++k) {
                        tk[k] = 0;
                        xd[k] = yd[k] = zd[k] = hd[k] = 0.0;
                        if (cb0 + 64 * k < total) {          // uniform
                            const int32_t f = max(wave_incl_max(mymark[64 * k + lane]), carry);
                            carry = __builtin_amdgcn_readlane(f, 63);
                            tk[k] = cb0 + 64 * k + (int32_t)lane + f;
                            const uint32_t t = (uint32_t)min(max(tk[k], 0), (int32_t)(ng - 1));
                            xd[k] = at32(xs, t);
                            yd[k] = at32(ys, t);
                            zd[k] = at32(zs, t);
                            hd[k] = at32(hs, t);
                        }
                        const int32_t nk = total - (cb0 + 64 * k);
                        vm[k] = nk >= 64 ? ~0ull : (nk > 0 ? (1ull << nk) - 1 : 0ull);
                    }
                    // (empty statements that take the loaded values keep
                    // the conversions, and their waits, behind the last load)
#pragma unroll
                    for (int k = 0; k < kHold; ++k) asm volatile("" : "+v"(hd[k]));
                    pre_rec ck[kHold];
                    float ak[kHold], bk[kHold];
#pragma unroll
                    for (int k = 0; k < kHold; ++k) {
                        ck[k].h = (float)hd[k];
                        if constexpr (kPre) {
                            ck[k].x = (float)(xd[k] - O[0]);
                            ck[k].y = (float)(yd[k] - O[1]);
                            ck[k].z = (float)(zd[k] - O[2]);
                            const float m = ck[k].tol();
                            ak[k] = cb0 + 64 * k + (int32_t)lane < total ? ck[k].a() - m : __builtin_inff();
                            bk[k] = 2.0f * m;
                        }
                    }
                    for (int L = lead; L < lead + nrun; ++L) {
                        // target L (uniform) against the chunk: the lanes
                        // with a hit as a mask a batch
                        unsigned long long mk[kHold];
                        const int64_t sL = g0 + L;
                        if constexpr (kPre) {
                            const pre_rec qi = mytq[L];
                            const pre_cut ci = mytc[L];
                            float t[kHold];
                            unsigned long long any = 0;
#pragma unroll
                            for (int k = 0; k < kHold; ++k) {
                                t[k] = __builtin_fmaf(-qi.h, ck[k].h,
                                    __builtin_fmaf(-qi.z, ck[k].z, __builtin_fmaf(-qi.y, ck[k].y,
                                    __builtin_fmaf(-qi.x, ck[k].x, ak[k]))));
                                mk[k] = __builtin_amdgcn_ballot_w64(!(t[k] >= ci.maybe));
                                any |= mk[k];
                            }
                            if (!any) continue;
                            // undecided pairs: the predicate itself
                            unsigned long long un = 0;
#pragma unroll
                            for (int k = 0; k < kHold; ++k)
                                un |= mk[k] & ~__builtin_amdgcn_ballot_w64(t[k] + bk[k] < ci.sure);
                            if (un) {
                                int64_t sq = sL;
                                asm volatile("" : "+s"(sq));          // (nor for this)
#pragma unroll
                                for (int k = 0; k < kHold; ++k) {
                                    int32_t q = tk[k];
                                    asm volatile("" : "+v"(q));   // (no addresses kept for this)
                                    q = min(max(q, 0), (int32_t)(ng - 1));
                                    const bool pr = nbr_pred(xs[sq], ys[sq], zs[sq], (float)hs[sq],
                                                             xs[q], ys[q], zs[q], hs[q]);
                                    mk[k] &= __builtin_amdgcn_ballot_w64(pr) & vm[k];
                                }
                            }
                        } else {
                            const target_rec ti = mytp[L];
#pragma unroll
                            for (int k = 0; k < kHold; ++k) {
                                mk[k] = 0;
                                if (cb0 + 64 * k < total)              // uniform
                                    mk[k] = __builtin_amdgcn_ballot_w64(nbr_pred_f(
                                        ti.x, ti.y, ti.z, ti.h, xd[k], yd[k], zd[k], ck[k].h)) & vm[k];
                            }
                        }
                        int32_t c = __builtin_amdgcn_readlane(mine, L);
#pragma unroll
                        for (int k = 0; k < kHold; ++k) {
                            // the target itself is looked for only in
                            // batches with a hit
                            if (mk[k] == 0) continue;
                            const unsigned long long mask =
                                mk[k] & ~__builtin_amdgcn_ballot_w64(tk[k] == (int32_t)sL);
                            // a full slot's last entry takes what does not
                            // fit: the row is searched again then
                            const uint32_t pos = min((uint32_t)c + (uint32_t)rank_below(mask),
                                                     (uint32_t)L * kSlot + (kSlot - 1));
                            if (__builtin_amdgcn_inverse_ballot_w64(mask)) wslots[pos] = tk[k];
                            c += __builtin_popcountll(mask);
                        }
                        // lane L's count := c (one lane written, whatever the
                        // execution mask)
                        c = __builtin_amdgcn_readfirstlane(c);
                        asm volatile("v_writelane_b32 %0, %1, m0" : "+v"(mine) : "s"(c), "{m0}"(L));
                    }
                }
            }
        }
    }
    if (live) cnt[s] = mine - (int32_t)lane * kSlot;
}

template <int NT>
__global__ __launch_bounds__(kBlock, NT >= kPreMin ? 8 : 6) void k_nbr_search(
    const sg_grid_dev* __restrict__ g, int64_t ng, const double* __restrict__ xs,
    const double* __restrict__ ys, const double* __restrict__ zs, const double* __restrict__ hs,
    const int64_t* __restrict__ off, const int32_t* __restrict__ perm,
    const int32_t* __restrict__ key, int32_t* __restrict__ cnt, int32_t* __restrict__ slots) {
    // first target slot of this wavefront (uniform: held in a scalar
    // register).  The XCDs take chunks of 16 consecutive workgroups in
    // turn: the work per slot varies across the collision, and handing
    // each XCD one contiguous share of the slots left some XCDs busy after
    // the others had drained (stage 1.83 -> 1.64 ms at 1M gas), while
    // plain launch order spreads neighbouring targets over all 8 L2s
    // (1.5x the fetched bytes of chunks of 16, at the same time).
    const int32_t w = __builtin_amdgcn_readfirstlane(
        (int32_t)(xcd_chunk_block(blockIdx.x, gridDim.x, 16) * kWaves + (threadIdx.x >> 6)));
    nbr_search_wave<NT>(g, ng, xs, ys, zs, hs, off, perm, key, cnt, slots, w);
}

// Move every target's slot to its CSR row, which starts at nbr_off[s - off0]
// (or search again into the row when the slot was too short).  Wavefront w
// takes targets kCompact w .. kCompact w + kCompact - 1, 64 / kCompact lanes
// each; a target with more than kSlot hits is searched again by the whole
// wavefront.
// Bound by memory once the loads of a whole row are in flight together and
// the scalar loads of every target's count and offset, one after the other
// in search of an overflowed slot, are a ballot: 182 -> 97 us at 1048576
// targets (about 0.5 GB), with 8 / 16 targets a wavefront 120 / 172.
constexpr int kCompact = 4;
constexpr int kCompactLanes = 64 / kCompact;
constexpr int kMove = kSlot / kCompactLanes;      // entries a lane: one pass a row
static_assert(kMove * kCompactLanes == kSlot, "a slot in one pass");

__device__ __attribute__((always_inline)) inline void nbr_copy_wave(
    const sg_grid_dev* __restrict__ g, int64_t ng, const double* __restrict__ xs,
    const double* __restrict__ ys, const double* __restrict__ zs, const double* __restrict__ hs,
    const int64_t* __restrict__ off, const int32_t* __restrict__ cnt,
    const int32_t* __restrict__ slots, const int64_t* nbr_off, int64_t off0,
    int32_t* __restrict__ nbr_idx, int64_t w) {
    const unsigned lane = threadIdx.x & 63;
    const int64_t s0 = w * kCompact;
    if (s0 >= ng) return;
    const int64_t s = s0 + lane / kCompactLanes;
    const int32_t c = s < ng ? cnt[s] : 0;
    const unsigned long long over = __ballot(c > kSlot);
    {
        const int32_t n = c > kSlot ? 0 : c;
        const int32_t* const from = slots + s * kSlot;
        int32_t* const dst = nbr_idx + nbr_off[(s < ng ? s : s0) - off0];
        const int32_t k = lane % kCompactLanes;
        int32_t v[kMove];
#pragma unroll
        for (int i = 0; i < kMove; ++i)
            if (k + i * kCompactLanes < n) v[i] = from[k + i * kCompactLanes];
#pragma unroll
        for (int i = 0; i < kMove; ++i)
            if (k + i * kCompactLanes < n) dst[k + i * kCompactLanes] = v[i];
    }
    if (over == 0) return;
    for (int j = 0; j < kCompact; ++j) {
        if (!((over >> (j * kCompactLanes)) & 1ull)) continue;
        const int64_t sj = s0 + j;
        const int64_t to = nbr_off[sj - off0];
        int64_t q = 0;
        nbr_scan(g, ng, sj, lane, xs, ys, zs, hs, off,
                 [&](unsigned long long mask, int64_t t, bool ok) {
                     if (ok) nbr_idx[to + q + rank_below(mask)] = (int32_t)t;
                     q += __builtin_popcountll(mask);
                 });
    }
}

// Up to this many targets, a workgroup of the copy adds up the counts before
// its own targets itself (at most 64 KB from L2) and writes their offsets:
// no scan and no check of their own (three launches and one).  Stage: 1009
// targets 31 -> 23 us, 4096 39 -> 33, 9001 56 -> 54.
constexpr int64_t kOwnScan = 16384;

__global__ __launch_bounds__(kBlock) void k_nbr_compact_own(
    sg_grid_dev* __restrict__ g, int64_t ng, const double* __restrict__ xs,
    const double* __restrict__ ys, const double* __restrict__ zs, const double* __restrict__ hs,
    const int64_t* __restrict__ off, const int32_t* __restrict__ cnt,
    const int32_t* __restrict__ slots, int64_t nnz_cap, int64_t* __restrict__ nbr_off,
    int32_t* __restrict__ nbr_idx) {
    constexpr int kPer = kWaves * kCompact;        // targets of a workgroup
    __shared__ int64_t s_off[kPer + 1];
    __shared__ int64_t s_w[kWaves];
    if (g->err & SGE_SORT_FATAL) {
        if (blockIdx.x == 0 && threadIdx.x == 0) g->nnz = 0;
        return;
    }
    const int tid = threadIdx.x;
    const unsigned lane = tid & 63;
    const int first = blockIdx.x * kPer;
    int64_t sum = 0;
    for (int k = tid; k < first; k += kBlock) sum += cnt[k];
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    if (lane == 0) s_w[tid >> 6] = sum;
    __syncthreads();
    if (tid < 64) {
        int64_t base = 0;
        for (int w = 0; w < kWaves; ++w) base += s_w[w];
        const int64_t c = (int)lane < kPer && first + (int)lane < ng ? cnt[first + lane] : 0;
        int64_t incl = c;
        for (int o = 1; o < kPer; o <<= 1) {
            const int64_t t = __shfl_up(incl, o, 64);
            if ((int)lane >= o) incl += t;
        }
        if ((int)lane < kPer) {
            s_off[lane] = base + incl - c;
            if (first + (int)lane < ng) nbr_off[first + lane] = base + incl - c;
            if ((int)lane == kPer - 1) s_off[kPer] = base + incl;
        }
    }
    __syncthreads();
    const int64_t end = s_off[kPer];
    // the last workgroup knows the total
    if (blockIdx.x == gridDim.x - 1 && tid == 0) {
        nbr_off[ng] = end;
        nbr_check_total(g, end, nnz_cap);
    }
    if (end > nnz_cap) return;                     // rows past the capacity are not written
    nbr_copy_wave(g, ng, xs, ys, zs, hs, off, cnt, slots, s_off, first, nbr_idx,
                  (int64_t)blockIdx.x * kWaves + (tid >> 6));
}

__global__ __launch_bounds__(kBlock) void k_nbr_compact(
    const sg_grid_dev* __restrict__ g, int64_t ng, const double* __restrict__ xs,
    const double* __restrict__ ys, const double* __restrict__ zs, const double* __restrict__ hs,
    const int64_t* __restrict__ off, const int32_t* __restrict__ cnt,
    const int32_t* __restrict__ slots, const int64_t* __restrict__ nbr_off,
    int32_t* __restrict__ nbr_idx) {
    if (g->err & (SGE_SORT_FATAL | SGE_NNZ)) return;
    const int64_t w = (int64_t)blockIdx.x * kWaves + (threadIdx.x >> 6);
    nbr_copy_wave(g, ng, xs, ys, zs, hs, off, cnt, slots, nbr_off, 0, nbr_idx, w);
}

// ----------------------------------------------------- all systems at once --
// (see sg_seg in sg_internal.h)

template <int NT>
__global__ __launch_bounds__(kBlock, NT >= kPreMin ? 8 : 6) void k_seg_nbr_search(
    const sg_seg_sys* __restrict__ sys, const int64_t* __restrict__ pfx, int nsys) {
    int64_t lb;
    const sg_seg_sys& S = sys[sg_seg_find(pfx, nsys, blockIdx.x, &lb)];
    const int32_t w = __builtin_amdgcn_readfirstlane((int32_t)(lb * kWaves + (threadIdx.x >> 6)));
    const sg_sph_bufs& b = S.sph;
    nbr_search_wave<NT>(S.g, S.ng, b.xs, b.ys, b.zs, b.hs, S.off, b.perm, S.key, S.ncnt, S.slots,
                        w);
}

__global__ void k_seg_nbr_check(const sg_seg_sys* __restrict__ sys, int nsys) {
    for (int k = threadIdx.x; k < nsys; k += blockDim.x)
        if (sys[k].ng > 0)
            nbr_check_total(sys[k].g, sys[k].sph.nbr_off[sys[k].ng], sys[k].nnz_cap);
}

__global__ __launch_bounds__(kBlock) void k_seg_nbr_compact(const sg_seg_sys* __restrict__ sys,
                                                            const int64_t* __restrict__ pfx,
                                                            int nsys) {
    int64_t lb;
    const sg_seg_sys& S = sys[sg_seg_find(pfx, nsys, blockIdx.x, &lb)];
    const sg_sph_bufs& b = S.sph;
    if (S.g->err & (SGE_SORT_FATAL | SGE_NNZ)) return;
    nbr_copy_wave(S.g, S.ng, b.xs, b.ys, b.zs, b.hs, S.off, S.ncnt, S.slots, b.nbr_off, 0,
                  const_cast<int32_t*>(b.nbr_idx), lb * kWaves + (threadIdx.x >> 6));
}

inline unsigned waves_grid(int64_t n) {
    int64_t b = (n + kWaves - 1) / kWaves;
    return (unsigned)(b < 1 ? 1 : b);
}

}  // namespace

// Targets per wavefront.  Few targets per wavefront give many short
// wavefronts: at a few thousand targets the stage is the latency of one
// wavefront's serial walk over its targets' levels, rows and passes.  Many
// share the set-up of a run's boxes and each candidate load among its
// targets, which is what counts once the wavefronts fill the chip.  Stage
// (search, scan, check, copy) in us with 32 / 16 / 8 / 4 / 2 / 1 targets: 1009
// targets 112 / 83 / 61 / 44 / 27 / 20; 9001: 170 / 100 / 67 / 58 / 52 / 47;
// 14000: 192 / 116 / 82 / 68 / 67 / 65; 20000: 202 / 125 / 92 / 81 / 71 / 80;
// 30011: 161 / 106 / 83 / 77 / 86 / 105; 45000: 146 / 100 / 87 / 91 / 106 /
// 137; 100000: 163 / 129 / 132 / 151 / 192 / 263; 131071: 166 / 152 / 151 /
// 178; 262144: 232 / 228 / 251 / 318; 400000: 320 / 315 / 363; 524288: 390 /
// 400 / 463; 1048576: 696 / 752 / 865.
int sg_nbr_targets(int64_t ng) {
    if (ng >= 450000) return 32;
    if (ng >= 120000) return 16;
    if (ng >= 40000) return 8;
    if (ng >= 25000) return 4;
    return ng >= 16000 ? 2 : 1;
}

namespace {
template <typename F>
void with_targets(int nt, F&& f) {
    switch (nt) {
        case 1: f(std::integral_constant<int, 1>()); break;
        case 2: f(std::integral_constant<int, 2>()); break;
        case 4: f(std::integral_constant<int, 4>()); break;
        case 8: f(std::integral_constant<int, 8>()); break;
        case 16: f(std::integral_constant<int, 16>()); break;
        default: f(std::integral_constant<int, 32>()); break;
    }
}
}  // namespace

void sg_seg_launch_nbr_search(const sg_seg& s, hipStream_t st) {
    if (s.nblk[SG_SEG_NBR] == 0) return;
    with_targets(s.nbr_targets, [&](auto nt) {
        hipLaunchKernelGGL((k_seg_nbr_search<decltype(nt)::value>),
                           dim3((unsigned)s.nblk[SG_SEG_NBR]), dim3(kBlock), 0, st, s.sys,
                           s.pfx + SG_SEG_NBR * (s.nsys + 1), s.nsys);
    });
}

void sg_seg_launch_nbr_finish(const sg_seg& s, hipStream_t st) {
    if (s.nblk[SG_SEG_CPT] == 0) return;
    hipLaunchKernelGGL(k_seg_nbr_check, dim3(1), dim3(64), 0, st, s.sys, s.nsys);
    hipLaunchKernelGGL(k_seg_nbr_compact, dim3((unsigned)s.nblk[SG_SEG_CPT]), dim3(kBlock), 0, st,
                       s.sys, s.pfx + SG_SEG_CPT * (s.nsys + 1), s.nsys);
}

int64_t sg_compact_blocks(int64_t ng) {
    const int64_t per = (int64_t)kWaves * kCompact;
    return (ng + per - 1) / per;
}

int64_t sg_nbr_blocks(int64_t ng, int nt) {
    const int64_t per = (int64_t)kWaves * nt;
    return (ng + per - 1) / per;
}

size_t sg_nbr_slot_bytes(int64_t ng) { return 4 * (size_t)kSlot * (size_t)(ng > 0 ? ng : 0); }

void sg_launch_nbr_search(const sg_grid_dev* g, int64_t ng, const double* xs, const double* ys,
                          const double* zs, const double* hs, const int64_t* off,
                          const int32_t* perm, const int32_t* key, int32_t* cnt, int32_t* slots,
                          hipStream_t st) {
    const int targets = sg_nbr_targets(ng);
    with_targets(targets, [&](auto nt) {
        hipLaunchKernelGGL((k_nbr_search<decltype(nt)::value>),
                           dim3(waves_grid((ng + targets - 1) / targets)), dim3(kBlock), 0, st, g,
                           ng, xs, ys, zs, hs, off, perm, key, cnt, slots);
    });
}

void sg_launch_nbr_finish(sg_grid_dev* g, int64_t ng, const double* xs, const double* ys,
                          const double* zs, const double* hs, const int64_t* off,
                          const int32_t* cnt, const int32_t* slots, int64_t nnz_cap, void* scan,
                          int64_t* nbr_off, int32_t* nbr_idx, hipStream_t st) {
    const unsigned nb = waves_grid((ng + kCompact - 1) / kCompact);
    if (ng <= kOwnScan) {
        hipLaunchKernelGGL(k_nbr_compact_own, dim3(nb), dim3(kBlock), 0, st, g, ng, xs, ys, zs, hs,
                           off, cnt, slots, nnz_cap, nbr_off, nbr_idx);
        return;
    }
    sg_launch_scan(cnt, nbr_off, ng, nullptr, ng, scan, st, g, nnz_cap);
    hipLaunchKernelGGL(k_nbr_compact, dim3(nb), dim3(kBlock), 0, st, g, ng, xs, ys, zs, hs, off,
                       cnt, slots, nbr_off, nbr_idx);
}
