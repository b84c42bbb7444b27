// sg_sort.hip -- grid sorting of the gas (the SP kernel set of Sec. 3):
// smoothing-length levels and grid parameters, cell keys, per-cell counts
// and maximum h, prefix sums for cell offsets, stable reorder and gather of
// the sorted state.  Also the generic scan used for cell and CSR offsets,
// and a stable LSD radix sort producing a Morton order of all particles.
//
// Built with -ffp-contract=off: the key arithmetic must round exactly like
// the plain FP64 definition of the grid.
#include <type_traits>

#include "sg_internal.h"

namespace {

constexpr int kBlock = 256;

__device__ inline unsigned lane_id() { return threadIdx.x & 63; }

// 64-bit minimum and maximum over the 64 lanes by DPP row operations on the
// two 32-bit halves, with no chain of shuffles through LDS (Morton box,
// equal-key runs of an ensemble's key pass).  Every lane must be active;
// the result is uniform.  Controls: quad_perm
// [1,0,3,2] 0xb1, [2,3,0,1] 0x4e, row_half_mirror 0x141, row_mirror 0x140,
// row_bcast:15 0x142 (lane 15 of each row into the next row), row_bcast:31
// 0x143 (lane 31 into rows 2 and 3).
template <int kCtrl, int kRowMask = 0xf>
__device__ inline unsigned long long dpp_u64(unsigned long long old, unsigned long long v) {
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp((int)(unsigned)old, (int)(unsigned)v,
                                                              kCtrl, kRowMask, 0xf, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(
        (int)(unsigned)(old >> 32), (int)(unsigned)(v >> 32), kCtrl, kRowMask, 0xf, false);
    return ((unsigned long long)hi << 32) | lo;
}
template <bool kMax>
__device__ inline unsigned long long wave_ext_u64(unsigned long long v) {
    constexpr unsigned long long I = kMax ? 0ull : ~0ull;
    auto pick = [](unsigned long long a, unsigned long long b) { return (kMax ? b > a : b < a) ? b : a; };
    v = pick(v, dpp_u64<0xb1>(I, v));
    v = pick(v, dpp_u64<0x4e>(I, v));
    v = pick(v, dpp_u64<0x141>(I, v));
    v = pick(v, dpp_u64<0x140>(I, v));          // each row of 16: its extreme
    v = pick(v, dpp_u64<0x142, 0xa>(I, v));     // rows 1, 3: with rows 0, 2
    v = pick(v, dpp_u64<0x143, 0xc>(I, v));     // rows 2, 3: with rows 0, 1
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, 63);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), 63);
    return ((unsigned long long)hi << 32) | lo;
}
__device__ inline unsigned long long wave_min_u64(unsigned long long v) { return wave_ext_u64<false>(v); }
__device__ inline unsigned long long wave_max_u64(unsigned long long v) { return wave_ext_u64<true>(v); }
__device__ inline unsigned long long wave_sum_u64(unsigned long long v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
// Number of set bits of `mask` below this lane.
__device__ inline unsigned rank_below(unsigned long long mask) {
    return __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
}

__global__ void k_nbr_check(sg_grid_dev* g, const int64_t* __restrict__ nbr_off, int64_t ng,
                            int64_t nnz_cap) {
    if (threadIdx.x == 0) nbr_check_total(g, nbr_off[ng], nnz_cap);
}

// ------------------------------------------------------------------ scan --
constexpr int kScanItems = 8;
constexpr int kScanTile = kBlock * kScanItems;

__device__ inline int64_t scan_n(int64_t n_host, const int64_t* n_dev, int64_t cap) {
    const int64_t n = n_dev ? *n_dev : n_host;
    return n < cap ? n : cap;
}

__device__ inline void scan_reduce_tile(const int32_t* __restrict__ in, int64_t n, int64_t tile,
                                        int64_t* __restrict__ bsum) {
    const int64_t base = tile * kScanTile;
    int64_t s = 0;
    for (int k = 0; k < kScanItems; ++k) {
        int64_t i = base + k * kBlock + threadIdx.x;
        if (i < n) s += in[i];
    }
    s = (int64_t)wave_sum_u64((unsigned long long)s);
    __shared__ int64_t ws[kBlock / 64];
    if (lane_id() == 0) ws[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t t = 0;
        for (int w = 0; w < kBlock / 64; ++w) t += ws[w];
        bsum[tile] = t;
    }
}

__global__ __launch_bounds__(kBlock) void k_scan_reduce(const int32_t* __restrict__ in,
                                                        int64_t n_host,
                                                        const int64_t* __restrict__ n_dev,
                                                        int64_t cap,
                                                        int64_t* __restrict__ bsum) {
    scan_reduce_tile(in, scan_n(n_host, n_dev, cap), blockIdx.x, bsum);
}

// Exclusive scan of the block sums in place; out[n] = total.  256 threads,
// 4 sums each per pass: one wavefront per SIMD, so the block also finds
// room on CUs that another kernel's workgroups mostly fill.
__device__ inline void scan_bsums_block(int64_t* __restrict__ bsum, int64_t n,
                                        int64_t* __restrict__ out) {
    const int64_t nb = (n + kScanTile - 1) / kScanTile;
    __shared__ int64_t buf[256];
    __shared__ int64_t carry;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int64_t c0 = 0; c0 < nb; c0 += 1024) {
        const int64_t i0 = c0 + 4 * (int64_t)threadIdx.x;
        int64_t v[4];
        int64_t tsum = 0;
        for (int k = 0; k < 4; ++k) {
            v[k] = i0 + k < nb ? bsum[i0 + k] : 0;
            tsum += v[k];
        }
        buf[threadIdx.x] = tsum;
        __syncthreads();
        for (int o = 1; o < 256; o <<= 1) {       // Hillis-Steele inclusive scan
            int64_t t = threadIdx.x >= (unsigned)o ? buf[threadIdx.x - o] : 0;
            __syncthreads();
            buf[threadIdx.x] += t;
            __syncthreads();
        }
        int64_t run = carry + buf[threadIdx.x] - tsum;
        for (int k = 0; k < 4; ++k) {
            if (i0 + k < nb) bsum[i0 + k] = run;
            run += v[k];
        }
        __syncthreads();
        if (threadIdx.x == 0) carry += buf[255];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[n] = carry;
}

__global__ __launch_bounds__(256) void k_scan_bsums(int64_t* __restrict__ bsum, int64_t n_host,
                                                    const int64_t* __restrict__ n_dev,
                                                    int64_t cap, int64_t* __restrict__ out) {
    scan_bsums_block(bsum, scan_n(n_host, n_dev, cap), out);
}

// before: sum of the tiles before this one; returns this tile's sum.
__device__ inline int64_t scan_down_tile(const int32_t* __restrict__ in, int64_t* __restrict__ out,
                                         int64_t n, int64_t tile, int64_t before) {
    const int64_t base = tile * kScanTile;
    if (base >= n) return 0;
    const int64_t i0 = base + (int64_t)threadIdx.x * kScanItems;
    int64_t v[kScanItems];
    int64_t tsum = 0;
    for (int k = 0; k < kScanItems; ++k) {
        v[k] = (i0 + k < n) ? in[i0 + k] : 0;
        tsum += v[k];
    }
    // exclusive scan of the thread sums across the block
    int64_t incl = tsum;
    for (int o = 1; o < 64; o <<= 1) {
        int64_t t = __shfl_up(incl, o, 64);
        if (lane_id() >= (unsigned)o) incl += t;
    }
    __shared__ int64_t wtot[kBlock / 64];
    if (lane_id() == 63) wtot[threadIdx.x >> 6] = incl;
    __syncthreads();
    int64_t wbase = 0;
    for (int w = 0; w < (int)(threadIdx.x >> 6); ++w) wbase += wtot[w];
    int64_t run = before + wbase + incl - tsum;
    for (int k = 0; k < kScanItems; ++k) {
        if (i0 + k < n) out[i0 + k] = run;
        run += v[k];
    }
    int64_t total = 0;
    for (int w = 0; w < kBlock / 64; ++w) total += wtot[w];
    return total;
}

__global__ __launch_bounds__(kBlock) void k_scan_down(const int32_t* __restrict__ in,
                                                      int64_t* __restrict__ out, int64_t n_host,
                                                      const int64_t* __restrict__ n_dev,
                                                      int64_t cap,
                                                      const int64_t* __restrict__ bsum) {
    scan_down_tile(in, out, scan_n(n_host, n_dev, cap), blockIdx.x, bsum[blockIdx.x]);
}

// The same without k_scan_bsums, for up to kScanOwn tiles: a workgroup adds
// up the sums of the tiles before it itself (8 KB from L2 at most), and the
// last one knows the total.  chk: the total is that of the neighbour lists,
// whose check needs no launch of its own then.
constexpr int64_t kScanOwn = 1024;
__global__ __launch_bounds__(kBlock) void k_scan_down_own(
    const int32_t* __restrict__ in, int64_t* __restrict__ out, int64_t n_host,
    const int64_t* __restrict__ n_dev, int64_t cap, const int64_t* __restrict__ bsum,
    sg_grid_dev* chk, int64_t nnz_cap) {
    const int64_t n = scan_n(n_host, n_dev, cap), tile = blockIdx.x;
    const int64_t tiles = n > 0 ? (n + kScanTile - 1) / kScanTile : 1;
    if (tile >= tiles) return;
    __shared__ int64_t s_b[kBlock / 64];
    int64_t b = 0;
    for (int64_t k = threadIdx.x; k < tile; k += kBlock) b += bsum[k];
    b = (int64_t)wave_sum_u64((unsigned long long)b);
    if (lane_id() == 0) s_b[threadIdx.x >> 6] = b;
    __syncthreads();
    b = 0;
    for (int w = 0; w < kBlock / 64; ++w) b += s_b[w];
    const int64_t total = b + scan_down_tile(in, out, n, tile, b);
    if (tile != tiles - 1 || threadIdx.x != 0) return;
    out[n] = total;
    if (chk) nbr_check_total(chk, total, nnz_cap);
}

// ------------------------------------------------------------ grid rule --

__device__ inline bool finite_d(double v) { return __builtin_isfinite(v); }

// Exponent field of the smallest power of two >= h (2 + 2^-9), the cell side
// that a particle asks for.
__device__ inline uint32_t side_exponent(double h) {
    const unsigned long long b =
        (unsigned long long)__builtin_bit_cast(long long, h * (2.0 + 0x1p-9));
    return (uint32_t)(b >> 52) + ((b & 0x000fffffffffffffull) ? 1u : 0u);
}

// First level l with L0 * 2^l >= h (2 + 2^-9); -1 beyond SG_MAXLEV.
__device__ inline int level_of(double h, double L0) {
    double t = h * (2.0 + 0x1p-9);
    double L = L0;
    int l = 0;
    while (L < t) {
        L *= 2.0;
        if (++l >= SG_MAXLEV) return -1;
    }
    return l;
}

// The grid's reduction inputs (lane l < SG_BINADES of a wavefront: binade l).
// They are reset when a state is bound, and by the pass that consumes them
// (grid_finish_wave) for the next build, so a build needs no launch for it;
// the gravity-order box likewise (by the gather in Morton order, in
// sg_grav.hip, after the Morton keys).
__device__ inline void grid_inputs_reset(sg_grid_dev* g, int l) {
    if (l == 0) {
        g->emin = ~0u;
        g->emax = 0u;
    }
    if (l < SG_BINADES) {
        for (int d = 0; d < 3; ++d) {
            g->bin[l].lo[d] = ~0ull;
            g->bin[l].hi[d] = 0ull;
        }
        g->bin[l].hmax = 0ull;
        g->bin[l].cnt = 0ull;
    }
}

__global__ void k_status_clear(sg_grid_dev* g, int record) {
    const int t = threadIdx.x;
    if (t == 0) {
        g->err = 0;
        g->need_cells = 0;
        g->need_nnz = 0;
    }
    if (!record) return;
    if (t == 0) {
        g->nnz = 0;
        g->M = 0;
        g->nlev = 0;
        g->ticket = 0;
    }
    if (t < SG_MAXLEV) {
        g->ncell[t] = 0;
        g->npart[t] = 0;
    }
    grid_inputs_reset(g, t);
    if (t < 3) {
        g->glo[t] = ~0ull;
        g->ghi[t] = 0ull;
    }
}

// Validity of the gas state, and bounds, maximum h and number of its
// particles by the binade of their cell side: which levels these are follows
// from the smallest one once all are in (grid_finish_wave), so one pass reads
// the state.  (A pass for the smallest h first: 21 us more at 1048576 gas
// particles, 8 at 131071, and a launch.)  Exponents that share an entry of
// the table differ by SG_BINADES or more, which is an error anyway.
//
// Items base + r * stride + threadIdx.x, r < nround, of a workgroup.  One LDS
// atomic per bound and particle (wavefront reductions per level present cost
// more), in kCopies copies of the table.  Bound by the workgroups' device
// atomics at the end, which meet at a few lines: see grid_blocks.
constexpr int kCopies = 16;
constexpr int kAhead = 4;                      // items in flight
__device__ inline void grid_levels_block(const double* __restrict__ x,
                                         const double* __restrict__ y,
                                         const double* __restrict__ z,
                                         const double* __restrict__ h, int64_t ng,
                                         sg_grid_dev* g, int64_t base, int64_t stride,
                                         int64_t nround) {
    __shared__ unsigned long long s_lo[3][SG_BINADES][kCopies], s_hi[3][SG_BINADES][kCopies];
    __shared__ unsigned long long s_hmax[SG_BINADES][kCopies], s_cnt[SG_BINADES][kCopies];
    __shared__ uint32_t s_e[2];
    static_assert(SG_BINADES * kCopies == kBlock, "a lane an entry");
    const int te = threadIdx.x / kCopies, tc = threadIdx.x % kCopies;
    for (int d = 0; d < 3; ++d) {
        s_lo[d][te][tc] = ~0ull;
        s_hi[d][te][tc] = 0ull;
    }
    s_hmax[te][tc] = s_cnt[te][tc] = 0ull;
    if (threadIdx.x == 0) {
        s_e[0] = ~0u;
        s_e[1] = 0u;
    }
    __syncthreads();
    bool bad = false;
    uint32_t mn = ~0u, mx = 0u;
    for (int64_t r = 0; r < nround; r += kAhead) {
        double hi[kAhead], p[kAhead][3];
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
            const int64_t i = (r + q) * stride + base + threadIdx.x;
            if (r + q >= nround || i >= ng) {
                hi[q] = -1.0;
                continue;
            }
            hi[q] = h[i];
            p[q][0] = x[i];
            p[q][1] = y[i];
            p[q][2] = z[i];
            if (!(hi[q] > 0.0)) bad = true;
        }
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
            if (!(hi[q] > 0.0)) continue;
            if (!finite_d(hi[q]) || !finite_d(p[q][0]) || !finite_d(p[q][1]) || !finite_d(p[q][2])) {
                bad = true;
                continue;
            }
            const uint32_t e = side_exponent(hi[q]);
            mn = e < mn ? e : mn;
            mx = e > mx ? e : mx;
            const int k = e % SG_BINADES;
            for (int d = 0; d < 3; ++d) {
                atomicMin(&s_lo[d][k][tc], sg_ord(p[q][d]));
                atomicMax(&s_hi[d][k][tc], sg_ord(p[q][d]));
            }
            atomicMax(&s_hmax[k][tc], sg_ord(hi[q]));
            atomicAdd(&s_cnt[k][tc], 1ull);
        }
    }
    if (bad) atomicOr(&g->err, SGE_NONFINITE);
    if (mn <= mx) {
        atomicMin(&s_e[0], mn);
        atomicMax(&s_e[1], mx);
    }
    __syncthreads();
    if (threadIdx.x == 0 && s_e[0] <= s_e[1]) {
        atomicMin(&g->emin, s_e[0]);
        atomicMax(&g->emax, s_e[1]);
    }
    // a lane a value: eight fields of each binade
    const int k = threadIdx.x / 8, f = threadIdx.x % 8;
    if (k >= SG_BINADES) return;
    unsigned long long c = 0;
    for (int q = 0; q < kCopies; ++q) c += s_cnt[k][q];
    if (c == 0) return;
    sg_grid_dev::binade& out = g->bin[k];
    if (f < 3) {
        unsigned long long v = ~0ull;
        for (int q = 0; q < kCopies; ++q) v = s_lo[f][k][q] < v ? s_lo[f][k][q] : v;
        atomicMin(&out.lo[f], v);
    } else if (f < 7) {
        unsigned long long v = 0ull;
        for (int q = 0; q < kCopies; ++q) {
            const unsigned long long w = f < 6 ? s_hi[f - 3][k][q] : s_hmax[k][q];
            v = w > v ? w : v;
        }
        atomicMax(f < 6 ? &out.hi[f - 3] : &out.hmax, v);
    } else {
        atomicAdd(&out.cnt, c);
    }
}

// A value that other workgroups wrote by device-scope atomics.
template <typename T>
__device__ inline T seen(T* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Cell sides L[l] = L0 2^(l + cell_scale_log2) (powers of two); the level of
// a particle depends on L0 only.  One wavefront, lane q < SG_BINADES binade q
// (all inputs in one round of loads; the levels one after the other on one
// thread took 7-12 us).
__device__ inline void grid_finish_wave(sg_grid_dev* g, int64_t cell_cap, double cell_scale) {
    const int q = threadIdx.x & 63;
    uint32_t err = seen(&g->err);
    const uint32_t emin = seen(&g->emin), emax = seen(&g->emax);
    unsigned long long np = 0, hb = 0, lo[3] = {0, 0, 0}, hi[3] = {0, 0, 0};
    if (q < SG_BINADES) {
        sg_grid_dev::binade& b = g->bin[q];
        np = seen(&b.cnt);
        hb = seen(&b.hmax);
        for (int d = 0; d < 3; ++d) {
            lo[d] = seen(&b.lo[d]);
            hi[d] = seen(&b.hi[d]);
        }
    }
    // (the loads of g->emin come back before any lane resets it)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    grid_inputs_reset(g, q);
    const int l = (int)(((uint32_t)q - emin) % SG_BINADES);     // the binade's level
    const bool mine = q < SG_BINADES && l < SG_MAXLEV;
    if (!(err & SGE_NONFINITE) && emax >= emin + SG_MAXLEV) {
        err |= SGE_LEVELS;
        if (q == 0) atomicOr(&g->err, SGE_LEVELS);
    }
    if (err & (SGE_NONFINITE | SGE_LEVELS)) {
        if (mine) {
            g->ncell[l] = 0;
            g->npart[l] = 0;
        }
        if (q == 0) {
            g->M = 0;
            g->nlev = 0;
        }
        return;
    }
    const double L0 = __builtin_bit_cast(double, (unsigned long long)emin << 52);
    double L = L0 * cell_scale;        // exact: cell_scale is 1/2, 1 or 2
    for (int k = 0; k < l && k < SG_MAXLEV; ++k) L *= 2.0;
    const double inv = 1.0 / L;        // exact: L is a power of two
    if (!mine) np = 0;
    int64_t nc = np ? 1 : 0, dim[3] = {0, 0, 0};
    double org[3] = {0.0, 0.0, 0.0};
    bool bad = false;
    if (np) {
        for (int d = 0; d < 3 && !bad; ++d) {
            const double plo = sg_unord(lo[d]), phi = sg_unord(hi[d]);
            org[d] = floor(plo * inv) * L;
            const double span = floor((phi - org[d]) * inv);
            bad = !(span < 2147483646.0);
            if (!bad) {
                dim[d] = (int64_t)span + 1;
                nc *= dim[d];
                bad = nc > 2147483647ll;
            }
        }
    }
    if (__ballot(bad)) nc = 0;
    // lane k: level k, for the offsets of the levels
    const int from = (int)((emin + (uint32_t)q) % SG_BINADES);
    const int64_t own = __shfl(nc, from, 64);
    const int any = __shfl((int)(np != 0), from, 64);          // (with all lanes active)
    const unsigned long long full = __ballot(q < SG_MAXLEV && any != 0);
    int64_t incl = own;
    for (int o = 1; o < SG_MAXLEV; o <<= 1) {
        const int64_t t = __shfl_up(incl, o, 64);
        if (q >= o) incl += t;
    }
    const int64_t M = __shfl(incl, SG_MAXLEV - 1, 64);
    const int64_t base = __shfl(incl - own, l, 64);
    if (mine) {
        g->invL[l] = inv;
        g->base[l] = base;
        g->hmaxlev[l] = np ? sg_unord(hb) : 0.0;
        g->npart[l] = np;
        g->ncell[l] = nc;
        for (int d = 0; d < 3; ++d) {
            g->dim[l][d] = dim[d];
            g->org[l][d] = org[d];
        }
    }
    const bool none = __ballot(bad) != 0ull || M > 2147483647ll;
    if (q != 0) return;
    g->L0 = L0;
    g->nlev = full ? 64 - __builtin_clzll(full) : 0;
    g->M = none ? 0 : M;
    if (none) {
        atomicOr(&g->err, SGE_GRID);
        return;
    }
    if (M > cell_cap) {
        atomicOr(&g->err, SGE_CELLS);
        g->need_cells = M;
    }
}

// Level bounds; the workgroup that ends last turns them into the grid.
__global__ __launch_bounds__(kBlock) void k_grid_levels(const double* __restrict__ x,
                                                        const double* __restrict__ y,
                                                        const double* __restrict__ z,
                                                        const double* __restrict__ h,
                                                        int64_t ng, sg_grid_dev* g,
                                                        int64_t cell_cap, double cell_scale,
                                                        int32_t* __restrict__ count,
                                                        unsigned long long* __restrict__ hmax,
                                                        int64_t nclear, unsigned nlev) {
    __shared__ int s_last;
    if (blockIdx.x >= nlev) {
        // small cell tables are cleared whole here, before their size is known
        const int64_t step = (int64_t)(gridDim.x - nlev) * kBlock;
        for (int64_t k = (int64_t)(blockIdx.x - nlev) * kBlock + threadIdx.x; k < nclear; k += step) {
            count[k] = 0;
            hmax[k] = 0ull;
        }
        return;
    }
    const int64_t stride = (int64_t)nlev * kBlock;
    grid_levels_block(x, y, z, h, ng, g, (int64_t)blockIdx.x * kBlock, stride,
                      (ng + stride - 1) / stride);
    // this workgroup's atomics (the only data handed over) have reached
    // memory before it draws its ticket
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) s_last = atomicAdd(&g->ticket, 1u) == nlev - 1;
    __syncthreads();
    if (!s_last || threadIdx.x >= 64) return;
    if (threadIdx.x == 0) atomicExch(&g->ticket, 0u);
    grid_finish_wave(g, cell_cap, cell_scale);
}

__device__ inline void cells_clear_block(const sg_grid_dev* g, int32_t* __restrict__ count,
                                         unsigned long long* __restrict__ hmax, int64_t b,
                                         int64_t nb) {
    if (g->err & SGE_SORT_FATAL) return;
    const int64_t M = g->M;
    for (int64_t k = b * kBlock + threadIdx.x; k < M; k += nb * kBlock) {
        count[k] = 0;
        hmax[k] = 0ull;
    }
}

__global__ __launch_bounds__(kBlock) void k_cells_clear(const sg_grid_dev* g,
                                                        int32_t* __restrict__ count,
                                                        unsigned long long* __restrict__ hmax) {
    cells_clear_block(g, count, hmax, blockIdx.x, gridDim.x);
}

// h > 0: orders as bits
__device__ inline unsigned long long h_bits(double h) {
    return (unsigned long long)__builtin_bit_cast(long long, h);
}

// Cell key of a particle of level l.
__device__ inline int32_t cell_key(const sg_grid_dev* g, int l, const double (&p)[3]) {
    int64_t c[3];
    for (int d = 0; d < 3; ++d) {
        double v = floor((p[d] - g->org[l][d]) * g->invL[l]);
        double top = (double)(g->dim[l][d] - 1);
        v = v < 0.0 ? 0.0 : (v > top ? top : v);
        c[d] = (int64_t)v;
    }
    return (int32_t)(g->base[l] + (c[2] * g->dim[l][1] + c[1]) * g->dim[l][0] + c[0]);
}

// Key and, in particle order, record of particle i (every lane of a quad
// calls this); returns the key, *hb the bits of h.
__device__ inline int32_t key_one(const double* __restrict__ x, const double* __restrict__ y,
                                  const double* __restrict__ z, const double* __restrict__ h,
                                  const double* __restrict__ m, int64_t i, bool valid,
                                  const sg_grid_dev* g, int32_t* __restrict__ key,
                                  sg_prec* __restrict__ pin, unsigned long long* hb = nullptr) {
    int32_t k = -1;
    sg_prec rec{};
    if (valid) {
        const double hi = h[i];
        const int l = level_of(hi, g->L0);
        const double p[3] = {x[i], y[i], z[i]};
        rec = sg_prec{p[0], p[1], p[2], hi, m[i], {0.0, 0.0, 0.0}};
        k = cell_key(g, l, p);
        key[i] = k;
        if (hb) *hb = h_bits(hi);
    }
    // the particle's record in particle order, for the gather
    uint4 v[4];
    rec_to(rec, v);
    quad_store64(pin, valid ? (int32_t)i : -1, v);
    return k;
}

// The same with the cell's count and maximum h, by atomics (an ensemble's).
// Every lane of the wavefront calls this (valid or not): the lanes that share
// the key of the first valid lane add their count and maximum h with one
// atomic each (clustered or coincident gas puts many particles of a
// wavefront in one cell); the others add their own.
__device__ inline void keys_count_wave(const double* __restrict__ x, const double* __restrict__ y,
                                       const double* __restrict__ z,
                                       const double* __restrict__ h,
                                       const double* __restrict__ m, int64_t i, bool valid,
                                       const sg_grid_dev* g, int32_t* __restrict__ key,
                                       int32_t* __restrict__ count,
                                       unsigned long long* __restrict__ hmax,
                                       sg_prec* __restrict__ pin) {
    unsigned long long hb = 0ull;
    const int32_t k = key_one(x, y, z, h, m, i, valid, g, key, pin, &hb);
    bool done = !valid;
    const unsigned long long act = __ballot(valid);
    if (act) {
        const int lead = __builtin_ctzll(act);
        const int32_t lk = __builtin_amdgcn_readlane(k, lead);
        const unsigned long long peers = __ballot(valid && k == lk);
        if (__builtin_popcountll(peers) > 1) {
            const bool mine = (peers >> lane_id()) & 1ull;
            const unsigned long long hm = wave_max_u64(mine ? hb : 0ull);
            if ((int)lane_id() == lead) {
                atomicAdd(&count[lk], (int32_t)__builtin_popcountll(peers));
                atomicMax(&hmax[lk], hm);
            }
            done = done || mine;
        }
    }
    if (!done) {
        atomicAdd(&count[k], 1);
        atomicMax(&hmax[k], hb);
    }
}

// Keys and records; the counts and maxima of the cells are left to the gather
// (cell_stats), where particles of a cell lie side by side.
__global__ __launch_bounds__(kBlock) void k_gas_keys(const double* __restrict__ x,
                                                     const double* __restrict__ y,
                                                     const double* __restrict__ z,
                                                     const double* __restrict__ h,
                                                     const double* __restrict__ m, int64_t ng,
                                                     const sg_grid_dev* g,
                                                     int32_t* __restrict__ key,
                                                     sg_prec* __restrict__ pin) {
    if (g->err & SGE_SORT_FATAL) return;
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    key_one(x, y, z, h, m, i, i < ng, g, key, pin);
}

// Counts and maximum h of the cells from the sorted keys: lanes of a
// wavefront hold consecutive slots s, so a cell's particles are neighbours
// and its last lane writes.  Cells that reach into another wavefront's slots
// add to the cleared tables.  (Atomics per particle from the key pass, in
// particle order, each went to a line of its own: with them that pass took
// 117 us at 1048576 particles, without 22, and the gather 45 instead of 33.)
__device__ inline void cell_stats(const uint32_t* __restrict__ keys, int64_t s, int64_t ng,
                                  double h, int32_t* __restrict__ count,
                                  unsigned long long* __restrict__ hmax) {
    const int lane = (int)lane_id();
    const bool live = s < ng;
    const uint32_t k = live ? keys[s] : ~0u;               // (keys are below 2^31)
    unsigned long long v = live ? h_bits(h) : 0ull;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t k2 = __shfl_up(k, o, 64);
        const unsigned long long v2 = __shfl_up(v, o, 64);
        if (lane >= o && k2 == k && v2 > v) v = v2;
    }
    uint32_t prev = __shfl_up(k, 1, 64), next = __shfl_down(k, 1, 64);
    if (lane == 0) prev = s > 0 && live ? keys[s - 1] : ~0u;
    if (lane == 63) next = s + 1 < ng ? keys[s + 1] : ~0u;
    const unsigned long long heads = __ballot(prev != k || lane == 0);
    const bool cut = __ballot(lane == 0 && prev == k) != 0;    // lane 0 is no first particle
    if (!live || (next == k && lane != 63)) return;
    const int first = 63 - __builtin_clzll(heads & (~0ull >> (63 - lane)));
    const int32_t n = lane - first + 1;
    if ((first == 0 && cut) || next == k) {
        atomicAdd(&count[k], n);
        atomicMax(&hmax[k], v);
    } else {
        count[k] = n;
        hmax[k] = v;
    }
}

// Slot s of the sorted state (every lane of a quad calls this).
__device__ inline void gather_put(int64_t s, bool live, const sg_prec& r, double* __restrict__ xs,
                                  double* __restrict__ ys, double* __restrict__ zs,
                                  double* __restrict__ hs, double* __restrict__ ms,
                                  sg_prec* __restrict__ prec, bool f32) {
    if (live) {
        xs[s] = r.x;
        ys[s] = r.y;
        zs[s] = r.z;
        hs[s] = r.h;
        ms[s] = r.m;
    }
    const int32_t to = live ? (int32_t)s : -1;
    if (f32) {
        uint4 w[2];
        rec_to(sg_prec32{r.x, r.y, r.z, (float)r.h, (float)r.m}, w);
        pair_store32(prec, to, w);
    } else {
        uint4 v[4];
        rec_to(r, v);
        quad_store64(prec, to, v);
    }
}

// Particles with a key below c, by bisection in the sorted keys.
__device__ inline int32_t key_rank(const uint32_t* __restrict__ keys, int64_t ng, int64_t c) {
    int32_t lo = 0, hi = (int32_t)ng;
    while (lo < hi) {
        const int32_t mid = (int32_t)(((uint32_t)lo + (uint32_t)hi) >> 1);
        if ((int64_t)keys[mid] < c) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// The stable order of the gas by cell key (ascending particle id inside a
// cell) comes from an LSD radix sort of the keys, sg_launch_gas_order;
// here the gather of the sorted state.  The particles arrive in any order,
// so the gather is random: it reads each particle's 64-byte record that
// the key pass wrote in particle order (one aligned line per particle)
// instead of five scattered doubles (five lines): at 1M gas its fetched
// bytes fell from 625 MB to about 130 MB.
// Every lane of a quad calls this; s >= ng: nothing to gather.
__device__ inline void gather_one(const int32_t* __restrict__ perm, int64_t s, int64_t ng,
                                  const sg_prec* __restrict__ pin, double* __restrict__ xs,
                                  double* __restrict__ ys, double* __restrict__ zs,
                                  double* __restrict__ hs, double* __restrict__ ms,
                                  sg_prec* __restrict__ prec, bool f32,
                                  const uint32_t* __restrict__ keys = nullptr,
                                  int32_t* __restrict__ count = nullptr,
                                  unsigned long long* __restrict__ hmax = nullptr) {
    const bool live = s < ng;
    uint4 v[4];
    quad_load64(pin, live ? perm[s] : 0, v);
    const sg_prec r = rec_of<sg_prec>(v);
    if (count) cell_stats(keys, s, ng, r.h, count, hmax);
    gather_put(s, live, r, xs, ys, zs, hs, ms, prec, f32);
}

__global__ __launch_bounds__(kBlock) void k_gather_gas(
    const int32_t* __restrict__ perm, int64_t ng, const sg_grid_dev* g,
    const sg_prec* __restrict__ pin, double* __restrict__ xs, double* __restrict__ ys,
    double* __restrict__ zs, double* __restrict__ hs, double* __restrict__ ms,
    sg_prec* __restrict__ prec, int f32, const uint32_t* __restrict__ keys,
    int32_t* __restrict__ count, unsigned long long* __restrict__ hmax) {
    if (g->err & SGE_SORT_FATAL) return;
    gather_one(perm, (int64_t)blockIdx.x * kBlock + threadIdx.x, ng, pin, xs, ys, zs, hs, ms, prec,
               f32 != 0, keys, count, hmax);
}

// The same, and in the workgroups after the first nbg the cell offsets, by
// bisection in the sorted keys (off[c] = particles with a key below c: what
// the scan of the counts gives) beside the gather instead of in three
// launches of a scan.
__global__ __launch_bounds__(kBlock) void k_gather_gas_off(
    const int32_t* __restrict__ perm, int64_t ng, const sg_grid_dev* g,
    const sg_prec* __restrict__ pin, double* __restrict__ xs, double* __restrict__ ys,
    double* __restrict__ zs, double* __restrict__ hs, double* __restrict__ ms,
    sg_prec* __restrict__ prec, int f32, int nbg, const uint32_t* __restrict__ keys,
    int64_t* __restrict__ off, int32_t* __restrict__ count,
    unsigned long long* __restrict__ hmax) {
    if (g->err & SGE_SORT_FATAL) return;
    if ((int)blockIdx.x < nbg) {
        gather_one(perm, (int64_t)blockIdx.x * kBlock + threadIdx.x, ng, pin, xs, ys, zs, hs, ms,
                   prec, f32 != 0, keys, count, hmax);
        return;
    }
    const int64_t M = g->M;
    for (int64_t c = (int64_t)(blockIdx.x - nbg) * kBlock + threadIdx.x; c <= M;
         c += (int64_t)(gridDim.x - nbg) * kBlock)
        off[c] = key_rank(keys, ng, c);
}

// ------------------------------------------------------ Morton ordering --

constexpr int kRadixItems = 16;
constexpr int kRadixTile = kBlock * kRadixItems;

// Fold one thread's bounds into the grid record: wavefront, then
// workgroup, then one global atomic per bound and workgroup (same-address
// atomics from every wavefront serialise in L2).
__device__ inline void gbox_fold(const unsigned long long (&mn)[3], const unsigned long long (&mx)[3],
                                 bool bad, sg_grid_dev* g) {
    __shared__ unsigned long long s_lo[3][kBlock / 64], s_hi[3][kBlock / 64];
    const int w = threadIdx.x >> 6;
    for (int d = 0; d < 3; ++d) {
        unsigned long long a = wave_min_u64(mn[d]), b = wave_max_u64(mx[d]);
        if (lane_id() == 0) {
            s_lo[d][w] = a;
            s_hi[d][w] = b;
        }
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        const int d = threadIdx.x;
        unsigned long long a = s_lo[d][0], b = s_hi[d][0];
        for (int k = 1; k < kBlock / 64; ++k) {
            a = s_lo[d][k] < a ? s_lo[d][k] : a;
            b = s_hi[d][k] > b ? s_hi[d][k] : b;
        }
        atomicMin(&g->glo[d], a);
        atomicMax(&g->ghi[d], b);
    }
    if (bad) atomicOr(&g->err, SGE_GNONFINITE);
}

__device__ inline void gbox_point(const double* __restrict__ x, const double* __restrict__ y,
                                  const double* __restrict__ z, int64_t i,
                                  unsigned long long (&mn)[3], unsigned long long (&mx)[3],
                                  bool& bad) {
    const double p[3] = {x[i], y[i], z[i]};
    for (int d = 0; d < 3; ++d) {
        if (!finite_d(p[d])) {
            bad = true;
            continue;
        }
        unsigned long long o = sg_ord(p[d]);
        mn[d] = o < mn[d] ? o : mn[d];
        mx[d] = o > mx[d] ? o : mx[d];
    }
}

__global__ __launch_bounds__(kBlock) void k_gbox(const double* __restrict__ x,
                                                 const double* __restrict__ y,
                                                 const double* __restrict__ z, int64_t n,
                                                 sg_grid_dev* g) {
    unsigned long long mn[3] = {~0ull, ~0ull, ~0ull}, mx[3] = {0, 0, 0};
    bool bad = false;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kBlock)
        gbox_point(x, y, z, i, mn, mx, bad);
    gbox_fold(mn, mx, bad, g);
}

__device__ inline uint32_t spread3(uint32_t v) {   // 10 bits -> every third bit
    v &= 0x3ff;
    v = (v | (v << 16)) & 0x030000ffu;
    v = (v | (v << 8)) & 0x0300f00fu;
    v = (v | (v << 4)) & 0x030c30c3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}

// Key of a point in the cube of side ext (1 + 2^-20) at lo: 10 bits an axis.
__device__ inline uint32_t morton_key(const double (&p)[3], const double (&lo)[3], double ext) {
    const double scale = ext > 0.0 ? 1024.0 / (ext * (1.0 + 0x1p-20)) : 0.0;
    uint32_t c[3];
    for (int d = 0; d < 3; ++d) {
        double v = (p[d] - lo[d]) * scale;
        v = v < 0.0 ? 0.0 : (v > 1023.0 ? 1023.0 : v);
        c[d] = (uint32_t)v;
    }
    return spread3(c[0]) | (spread3(c[1]) << 1) | (spread3(c[2]) << 2);
}

__device__ inline void morton_key_one(const double* __restrict__ x, const double* __restrict__ y,
                                      const double* __restrict__ z, int64_t i,
                                      const sg_grid_dev* g, uint32_t* __restrict__ keys) {
    double lo[3], ext = 0.0;
    for (int d = 0; d < 3; ++d) {
        lo[d] = sg_unord(g->glo[d]);
        double e = sg_unord(g->ghi[d]) - lo[d];
        ext = e > ext ? e : ext;
    }
    const double p[3] = {x[i], y[i], z[i]};
    keys[i] = morton_key(p, lo, ext);
}

__global__ __launch_bounds__(kBlock) void k_morton_keys(const double* __restrict__ x,
                                                        const double* __restrict__ y,
                                                        const double* __restrict__ z, int64_t n,
                                                        const sg_grid_dev* g,
                                                        uint32_t* __restrict__ keys) {
    int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    morton_key_one(x, y, z, i, g, keys);
}

// Morton keys have 30 bits: three passes of 10-bit digits.
constexpr int kRadixBits = 10;
constexpr int kBuckets = 1 << kRadixBits;
constexpr int kRadixPasses = 3;

// Digit histogram of one tile of kBlock * ITEMS keys, digit-major
// (hist[d * ntiles + tile], for a scan over it) or, ROWS, tile-major.
template <int ITEMS = kRadixItems, bool ROWS = false>
__device__ inline void radix_hist_tile(const uint32_t* __restrict__ keys, int64_t n, int shift,
                                       int64_t ntiles, int32_t* __restrict__ hist,
                                       int64_t tile) {
    __shared__ int32_t s_h[kBuckets];
    for (int t = threadIdx.x; t < kBuckets; t += kBlock) s_h[t] = 0;
    __syncthreads();
    const int64_t base = tile * (kBlock * ITEMS);
    for (int k = 0; k < ITEMS; ++k) {
        int64_t i = base + k * kBlock + threadIdx.x;
        if (i < n) atomicAdd(&s_h[(keys[i] >> shift) & (kBuckets - 1)], 1);
    }
    __syncthreads();
    for (int t = threadIdx.x; t < kBuckets; t += kBlock)
        hist[ROWS ? tile * kBuckets + t : (int64_t)t * ntiles + tile] = s_h[t];
}

__global__ __launch_bounds__(kBlock) void k_radix_hist(const uint32_t* __restrict__ keys,
                                                       int64_t n, int shift, int64_t ntiles,
                                                       int32_t* __restrict__ hist) {
    radix_hist_tile(keys, n, shift, ntiles, hist, blockIdx.x);
}

// Stable scatter: element order inside the tile is preserved within each
// digit.  A wavefront takes a contiguous quarter of the tile and counts its
// digits in an LDS column of its own, in order and without a barrier: the
// count it finds is the rank of an element among its digit's earlier ones in
// the quarter.  One barrier later the columns of the wavefronts before it
// are known.  Bound by latency (one load of every element in flight, then
// ITEMS rounds of ten ballots and an LDS exchange), not by memory; with
// chunks of kBlock elements shared by the wavefronts, three barriers and a
// load to wait for in every round, a pass of 8192 keys took 10.7 us where
// this takes 7.6, one of 131071 13.5 (10.6), one of 1048576 23.8 (20.5).
// vin == nullptr stands for the values 0, 1, 2, .. (the element indices).
// ROWS: first positions by digit in s_base (LDS) instead of offs.
template <int ITEMS = kRadixItems, bool ROWS = false>
__device__ inline void radix_scatter_tile(const uint32_t* __restrict__ kin,
                                          const int32_t* __restrict__ vin, int64_t n, int shift,
                                          int64_t ntiles, const int64_t* __restrict__ offs,
                                          uint32_t* __restrict__ kout,
                                          int32_t* __restrict__ vout, int64_t tile,
                                          const int32_t* s_base = nullptr) {
    // 8 KB of LDS: small enough to find room on CUs that a gravity kernel
    // mostly fills
    constexpr int kWaves = kBlock / 64;
    static_assert(64 * ITEMS < 65536, "counts of a quarter in 16 bits");
    __shared__ uint16_t s_cnt[kWaves][kBuckets];
    const int wave = threadIdx.x >> 6, lane = (int)lane_id();
    const int64_t base = tile * (kBlock * ITEMS) + wave * (64 * ITEMS) + lane;
    uint32_t key[ITEMS];
    int32_t val[ITEMS], rank[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int64_t i = base + 64 * k;
        key[k] = i < n ? kin[i] : 0u;
        val[k] = i < n ? (vin ? vin[i] : (int32_t)i) : 0;
    }
    uint16_t* const cnt = s_cnt[wave];
    for (int t = 2 * lane; t < kBuckets; t += 128) cnt[t] = cnt[t + 1] = 0;
    wave_sync();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const bool valid = base + 64 * k < n;
        const uint32_t d = (key[k] >> shift) & (kBuckets - 1);
        unsigned long long peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < kRadixBits; ++b) {
            const unsigned long long bb = __ballot((d >> b) & 1u);
            peers &= ((d >> b) & 1u) ? bb : ~bb;
        }
        const int r = (int)rank_below(peers);
        const int before = cnt[d];
        rank[k] = before + r;
        wave_sync();
        if (valid && r == 0) cnt[d] = (uint16_t)(before + __builtin_popcountll(peers));
        wave_sync();
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        if (base + 64 * k >= n) break;                     // (later elements lie further up)
        const uint32_t d = (key[k] >> shift) & (kBuckets - 1);
        int32_t pre = rank[k];
        for (int w = 0; w < wave; ++w) pre += s_cnt[w][d];
        const int64_t dest = (ROWS ? (int64_t)s_base[d] : offs[(int64_t)d * ntiles + tile]) + pre;
        kout[dest] = key[k];
        vout[dest] = val[k];
    }
}

__global__ __launch_bounds__(kBlock) void k_radix_scatter(
    const uint32_t* __restrict__ kin, const int32_t* __restrict__ vin, int64_t n, int shift,
    int64_t ntiles, const int64_t* __restrict__ offs, uint32_t* __restrict__ kout,
    int32_t* __restrict__ vout) {
    radix_scatter_tile(kin, vin, n, shift, ntiles, offs, kout, vout, blockIdx.x);
}

// One pass in two launches, for up to kRowTiles tiles: the histograms are
// stored tile after tile, and every workgroup of the scatter adds up the rows
// itself (4 KB a tile from L2; four digits a lane) instead of three launches
// of a scan: at 8192 keys a pass took 30 us, of which the scan 10 and the
// scatter's 16 rounds 18.  Tiles shrink with n to fewer rounds of more
// workgroups.  (Counting a pass's histograms in the scatter before it, by
// global additions into the destination's tile, saves that launch too, but
// cost more: a pass of 131071 keys 24.7 us against 10.6 + 4.8.)  With the
// launches saved by k_grid_levels (which finishes the grid and clears small
// tables) and k_gather_gas_off, the sort stage went from
// 107 to 48 us at 9001 gas particles, 136 to 70 at 65536, 198 to 123 at
// 131071 and 243 to 184 at 262144.
constexpr int64_t kRowTiles = 64;
template <int ITEMS>
__global__ __launch_bounds__(kBlock) void k_radix_hist_rows(const uint32_t* __restrict__ keys,
                                                            int64_t n, int shift,
                                                            int32_t* __restrict__ hist) {
    radix_hist_tile<ITEMS, true>(keys, n, shift, 0, hist, blockIdx.x);
}

template <int ITEMS>
__global__ __launch_bounds__(kBlock) void k_radix_scatter_rows(
    const uint32_t* __restrict__ kin, const int32_t* __restrict__ vin, int64_t n, int shift,
    int ntiles, const int32_t* __restrict__ hist, uint32_t* __restrict__ kout,
    int32_t* __restrict__ vout) {
    __shared__ int32_t s_base[kBuckets];
    __shared__ int32_t s_w[kBlock / 64];
    const int tile = blockIdx.x, tid = threadIdx.x;
    const int4* row = reinterpret_cast<const int4*>(hist) + tid;
    int4 tot = make_int4(0, 0, 0, 0), pre = tot;
#pragma unroll 8
    for (int t = 0; t < ntiles; ++t) {
        const int4 v = row[t * (kBuckets / 4)];
        const int m = t < tile ? -1 : 0;
        tot.x += v.x;
        tot.y += v.y;
        tot.z += v.z;
        tot.w += v.w;
        pre.x += v.x & m;
        pre.y += v.y & m;
        pre.z += v.z & m;
        pre.w += v.w & m;
    }
    const int32_t sum = tot.x + tot.y + tot.z + tot.w;
    int32_t incl = sum;
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t t = __shfl_up(incl, o, 64);
        if (lane_id() >= (unsigned)o) incl += t;
    }
    if (lane_id() == 63) s_w[tid >> 6] = incl;
    __syncthreads();
    int32_t first = incl - sum;
    for (int w = 0; w < tid >> 6; ++w) first += s_w[w];
    s_base[4 * tid] = first + pre.x;
    s_base[4 * tid + 1] = first + tot.x + pre.y;
    s_base[4 * tid + 2] = first + tot.x + tot.y + pre.z;
    s_base[4 * tid + 3] = first + tot.x + tot.y + tot.z + pre.w;
    // (radix_scatter_tile synchronises before it reads them)
    radix_scatter_tile<ITEMS, true>(kin, vin, n, shift, ntiles, nullptr, kout, vout, tile, s_base);
}

// ------------------------------------------------ a few thousand particles --
//
// Keys and all passes of their sort in one launch: a workgroup of 1024 lanes
// holds up to 4096 keys and indices in LDS.  A pass is radix_scatter_tile's,
// with sixteen wavefronts' columns of counts summed by the lanes (a digit
// each) instead of by another launch; bound by latency (barriers, LDS round
// trips, the ballots of one compute unit).  The general chains take eight
// launches (Morton order) and five (gas) that cost the host 4-6 us each.
// Measured: Morton order of 2552 particles 28 us in eight kernels, 22 in
// one; keys to sorted state of 1009 gas particles 23 us in six, 14 in two
// (sort stage 34 -> 26 us; 4096: 43 -> 40).  A step of 1009 + 1543 particles
// went from 148 to 117 us.  (Up to 8192 keys the order takes 39 us instead of
// 41, but sixteen steps of 4096 + 4096 took anything from 2.9 to 3.6 ms
// against 3.25: gravity then runs beside the gas sort's one workgroup.)
constexpr int kSmall = 4096;
constexpr int kSmallBlock = 1024;
constexpr int kSmallItems = kSmall / kSmallBlock;
struct small_lds {
    uint32_t key[kSmall];
    uint16_t idx[kSmall];
    uint16_t cnt[kSmallBlock / 64][kBuckets];
    int32_t first[kBuckets];
    int32_t wsum[kSmallBlock / 64];
};
static_assert(kBuckets == kSmallBlock, "a lane a digit");

// inclusive prefix sum over the wavefront (every lane active)
__device__ inline int32_t wave_incl_sum_dpp(int32_t v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr 1, 2, 4, 8
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast 15, 31
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
    return v;
}

// Stable order of L.key / L.idx [0, n) over `passes` digits.
__device__ inline void small_sort(small_lds& L, int n, int passes) {
    const int tid = threadIdx.x, w = tid >> 6, lane = (int)lane_id();
    const int items = (n + kSmallBlock - 1) / kSmallBlock;
    const int base = w * 64 * items + lane;
    uint16_t* const cnt = L.cnt[w];
    for (int pass = 0; pass < passes; ++pass) {
        const int shift = kRadixBits * pass;
        uint32_t key[kSmallItems];
        int32_t idx[kSmallItems], rank[kSmallItems];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kSmallItems; ++k) {
            if (k >= items) break;                         // uniform
            const int i = base + 64 * k;
            key[k] = i < n ? L.key[i] : 0u;
            idx[k] = i < n ? L.idx[i] : 0;
        }
        for (int t = 2 * lane; t < kBuckets; t += 128) cnt[t] = cnt[t + 1] = 0;
        wave_sync();
#pragma unroll
        for (int k = 0; k < kSmallItems; ++k) {
            if (k >= items) break;
            const bool valid = base + 64 * k < n;
            const uint32_t d = (key[k] >> shift) & (kBuckets - 1);
            unsigned long long peers = __ballot(valid);
#pragma unroll
            for (int b = 0; b < kRadixBits; ++b) {
                const unsigned long long bb = __ballot((d >> b) & 1u);
                peers &= ((d >> b) & 1u) ? bb : ~bb;
            }
            const int r = (int)rank_below(peers), before = cnt[d];
            rank[k] = before + r;
            wave_sync();
            if (valid && r == 0) cnt[d] = (uint16_t)(before + __builtin_popcountll(peers));
            wave_sync();
        }
        __syncthreads();
        int32_t sum = 0;                                   // digit tid
#pragma unroll
        for (int v = 0; v < kSmallBlock / 64; ++v) {
            const int32_t c = L.cnt[v][tid];
            L.cnt[v][tid] = (uint16_t)sum;
            sum += c;
        }
        const int32_t incl = wave_incl_sum_dpp(sum);
        if (lane == 63) L.wsum[w] = incl;
        __syncthreads();
        const int32_t ws = wave_incl_sum_dpp(lane < w ? L.wsum[lane] : 0);   // (w < 64)
        L.first[tid] = incl - sum + __builtin_amdgcn_readlane(ws, 63);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kSmallItems; ++k) {
            if (k >= items || base + 64 * k >= n) break;
            const uint32_t d = (key[k] >> shift) & (kBuckets - 1);
            const int dest = L.first[d] + cnt[d] + rank[k];
            L.key[dest] = key[k];
            L.idx[dest] = (uint16_t)idx[k];
        }
    }
    __syncthreads();
}

__global__ __launch_bounds__(kSmallBlock) void k_morton_small(const double* __restrict__ x,
                                                              const double* __restrict__ y,
                                                              const double* __restrict__ z, int n,
                                                              sg_grid_dev* g,
                                                              int32_t* __restrict__ order) {
    __shared__ small_lds L;
    __shared__ unsigned long long s_lo[3][kSmallBlock / 64], s_hi[3][kSmallBlock / 64];
    const int tid = threadIdx.x;
    unsigned long long mn[3] = {~0ull, ~0ull, ~0ull}, mx[3] = {0, 0, 0};
    bool bad = false;
    const int items = (n + kSmallBlock - 1) / kSmallBlock;
    double p[kSmallItems][3];
#pragma unroll
    for (int k = 0; k < kSmallItems; ++k) {
        if (k >= items) break;                             // uniform
        const int i = tid + k * kSmallBlock < n ? tid + k * kSmallBlock : 0;
        p[k][0] = x[i];
        p[k][1] = y[i];
        p[k][2] = z[i];
    }
#pragma unroll
    for (int k = 0; k < kSmallItems; ++k) {
        if (k >= items) break;
        for (int d = 0; d < 3; ++d) {                      // (a repeated point 0 does no harm)
            if (!finite_d(p[k][d])) {
                bad = true;
                continue;
            }
            const unsigned long long o = sg_ord(p[k][d]);
            mn[d] = o < mn[d] ? o : mn[d];
            mx[d] = o > mx[d] ? o : mx[d];
        }
    }
    if (bad) atomicOr(&g->err, SGE_GNONFINITE);
    for (int d = 0; d < 3; ++d) {
        const unsigned long long a = wave_min_u64(mn[d]), b = wave_max_u64(mx[d]);
        if (lane_id() == 0) {
            s_lo[d][tid >> 6] = a;
            s_hi[d][tid >> 6] = b;
        }
    }
    __syncthreads();
    double lo[3], ext = 0.0;
    for (int d = 0; d < 3; ++d) {
        unsigned long long a = s_lo[d][0], b = s_hi[d][0];
        for (int k = 1; k < kSmallBlock / 64; ++k) {
            a = s_lo[d][k] < a ? s_lo[d][k] : a;
            b = s_hi[d][k] > b ? s_hi[d][k] : b;
        }
        lo[d] = sg_unord(a);
        const double e = sg_unord(b) - lo[d];
        ext = e > ext ? e : ext;
    }
#pragma unroll
    for (int k = 0; k < kSmallItems; ++k) {
        if (k >= items) break;
        const int i = tid + k * kSmallBlock;
        if (i < n) {
            L.key[i] = morton_key(p[k], lo, ext);
            L.idx[i] = (uint16_t)i;
        }
    }
    small_sort(L, n, kRadixPasses);
    for (int i = tid; i < n; i += kSmallBlock) order[i] = L.idx[i];
}

// Cell keys, their stable order and the keys in it.
__global__ __launch_bounds__(kSmallBlock) void k_keys_small(
    const double* __restrict__ x, const double* __restrict__ y, const double* __restrict__ z,
    const double* __restrict__ h, int ng, const sg_grid_dev* g, int passes,
    int32_t* __restrict__ key, uint32_t* __restrict__ sorted, int32_t* __restrict__ perm) {
    __shared__ small_lds L;
    if (g->err & SGE_SORT_FATAL) return;
    const int tid = threadIdx.x;
    const int items = (ng + kSmallBlock - 1) / kSmallBlock;
    double p[kSmallItems][3], hi[kSmallItems];
#pragma unroll
    for (int k = 0; k < kSmallItems; ++k) {
        if (k >= items) break;                             // uniform
        const int i = tid + k * kSmallBlock < ng ? tid + k * kSmallBlock : 0;
        p[k][0] = x[i];
        p[k][1] = y[i];
        p[k][2] = z[i];
        hi[k] = h[i];
    }
#pragma unroll
    for (int k = 0; k < kSmallItems; ++k) {
        if (k >= items) break;
        const int i = tid + k * kSmallBlock;
        if (i < ng) {
            const int32_t c = cell_key(g, level_of(hi[k], g->L0), p[k]);
            key[i] = c;
            L.key[i] = (uint32_t)c;
            L.idx[i] = (uint16_t)i;
        }
    }
    small_sort(L, ng, passes);
    for (int i = tid; i < ng; i += kSmallBlock) {
        sorted[i] = L.key[i];
        perm[i] = L.idx[i];
    }
}

// k_gather_gas_off from the particle-order arrays.
__global__ __launch_bounds__(kBlock) void k_gather_gas_small(
    const int32_t* __restrict__ perm, int64_t ng, const sg_grid_dev* g,
    const double* __restrict__ x, const double* __restrict__ y, const double* __restrict__ z,
    const double* __restrict__ h, const double* __restrict__ m, double* __restrict__ xs,
    double* __restrict__ ys, double* __restrict__ zs, double* __restrict__ hs,
    double* __restrict__ ms, sg_prec* __restrict__ prec, int f32, int nbg,
    const uint32_t* __restrict__ keys, int64_t* __restrict__ off, int32_t* __restrict__ count,
    unsigned long long* __restrict__ hmax) {
    if (g->err & SGE_SORT_FATAL) return;
    if ((int)blockIdx.x < nbg) {
        const int64_t s = (int64_t)blockIdx.x * kBlock + threadIdx.x;
        const bool live = s < ng;
        const int32_t i = live ? perm[s] : 0;
        const sg_prec r{x[i], y[i], z[i], h[i], m[i], {0.0, 0.0, 0.0}};
        cell_stats(keys, s, ng, r.h, count, hmax);
        gather_put(s, live, r, xs, ys, zs, hs, ms, prec, f32 != 0);
        return;
    }
    const int64_t M = g->M;
    for (int64_t c = (int64_t)(blockIdx.x - nbg) * kBlock + threadIdx.x; c <= M;
         c += (int64_t)(gridDim.x - nbg) * kBlock)
        off[c] = key_rank(keys, ng, c);
}

// ---------------------------------------- Morton order, all systems at once --
// (see sg_seg in sg_internal.h).  The same stable order as the per-system
// sort: the same keys, digits and stable scatter.

__global__ __launch_bounds__(kBlock) void k_seg_gbox(const sg_seg_sys* __restrict__ sys,
                                                     const int64_t* __restrict__ pfx, int nsys) {
    int64_t lb;
    const sg_seg_sys& S = sys[sg_seg_find(pfx, nsys, blockIdx.x, &lb)];
    unsigned long long mn[3] = {~0ull, ~0ull, ~0ull}, mx[3] = {0, 0, 0};
    bool bad = false;
    const int64_t i = lb * kBlock + threadIdx.x;
    if (i < S.n) gbox_point(S.x, S.y, S.z, i, mn, mx, bad);
    gbox_fold(mn, mx, bad, S.g);
}

__global__ __launch_bounds__(kBlock) void k_seg_morton_keys(const sg_seg_sys* __restrict__ sys,
                                                            const int64_t* __restrict__ pfx,
                                                            int nsys) {
    int64_t lb;
    const sg_seg_sys& S = sys[sg_seg_find(pfx, nsys, blockIdx.x, &lb)];
    const int64_t i = lb * kBlock + threadIdx.x;
    if (i < S.n) morton_key_one(S.x, S.y, S.z, i, S.g, S.mk0);
}

// pass p reads buffer p & 1 and writes the other one; the last pass writes
// the values to the order
__global__ __launch_bounds__(kBlock) void k_seg_radix_hist(const sg_seg_sys* __restrict__ sys,
                                                           const int64_t* __restrict__ pfx,
                                                           int nsys, int pass) {
    int64_t tile;
    const sg_seg_sys& S = sys[sg_seg_find(pfx, nsys, blockIdx.x, &tile)];
    radix_hist_tile((pass & 1) ? S.mk1 : S.mk0, S.n, kRadixBits * pass, S.ntiles, S.mhist, tile);
}

__global__ __launch_bounds__(kBlock) void k_seg_radix_scatter(const sg_seg_sys* __restrict__ sys,
                                                              const int64_t* __restrict__ pfx,
                                                              int nsys, int pass) {
    int64_t tile;
    const sg_seg_sys& S = sys[sg_seg_find(pfx, nsys, blockIdx.x, &tile)];
    const bool odd = pass & 1;
    int32_t* vout = pass == kRadixPasses - 1 ? S.order : (odd ? S.mv0 : S.mv1);
    radix_scatter_tile(odd ? S.mk1 : S.mk0, pass == 0 ? nullptr : (odd ? S.mv1 : S.mv0), S.n, kRadixBits * pass,
                       S.ntiles, S.moffs, odd ? S.mk0 : S.mk1, vout, tile);
}

// Exclusive scan of one system's digit histogram (1024 * ntiles counts)
// into its offsets, one workgroup per system; offs[total] is not needed by
// the scatter and not written.  gas: the cell-key sort's histogram, else the
// Morton sort's.  256 lanes: the cell-key sort runs beside the persistent
// gravity kernel, and a 1024-lane workgroup (4 free wave slots on every
// SIMD of one CU) waited there for the gravity kernel to end (173 ms).
constexpr int kSegScanBlock = 256;
__global__ __launch_bounds__(kSegScanBlock) void k_seg_scan_hist(const sg_seg_sys* __restrict__ sys,
                                                                 int gas) {
    const sg_seg_sys& S = sys[blockIdx.x];
    const int32_t* hist = gas ? S.ghist : S.mhist;
    int64_t* offs = gas ? S.goffs : S.moffs;
    const int64_t n = (int64_t)kBuckets * (gas ? S.gntiles : S.ntiles);
    __shared__ int64_t s_w[kSegScanBlock / 64];
    __shared__ int64_t s_carry;
    if (threadIdx.x == 0) s_carry = 0;
    __syncthreads();
    constexpr int kItems = 4;
    for (int64_t c0 = 0; c0 < n; c0 += (int64_t)kSegScanBlock * kItems) {
        const int64_t i0 = c0 + (int64_t)threadIdx.x * kItems;
        int64_t v[kItems], tsum = 0;
        for (int k = 0; k < kItems; ++k) {
            v[k] = i0 + k < n ? hist[i0 + k] : 0;
            tsum += v[k];
        }
        int64_t incl = tsum;
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t t = __shfl_up(incl, o, 64);
            if (lane_id() >= (unsigned)o) incl += t;
        }
        if (lane_id() == 63) s_w[threadIdx.x >> 6] = incl;
        __syncthreads();
        int64_t wbase = s_carry;
        for (int w = 0; w < (int)(threadIdx.x >> 6); ++w) wbase += s_w[w];
        int64_t run = wbase + incl - tsum;
        for (int k = 0; k < kItems; ++k) {
            if (i0 + k < n) offs[i0 + k] = run;
            run += v[k];
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            int64_t t = 0;
            for (int w = 0; w < kSegScanBlock / 64; ++w) t += s_w[w];
            s_carry += t;
        }
        __syncthreads();
    }
}

// ----------------------------------------- gas sort, all systems at once --
// (see sg_seg in sg_internal.h): the per-system kernels' bodies; a system
// without gas is skipped, as the per-system build does.

__global__ __launch_bounds__(kBlock) void k_seg_grid_levels(const sg_seg_sys* __restrict__ sys,
                                                            const int64_t* __restrict__ pfx,
                                                            int nsys) {
    int64_t lb;
    const sg_seg_sys& S = sys[sg_seg_find(pfx, nsys, blockIdx.x, &lb)];
    grid_levels_block(S.x, S.y, S.z, S.h, S.ng, S.g, lb * kBlock, 0, 1);
}

__global__ void k_seg_grid_finish(const sg_seg_sys* __restrict__ sys) {
    const sg_seg_sys& S = sys[blockIdx.x];
    if (S.ng > 0) grid_finish_wave(S.g, S.cell_cap, S.cell_scale);
}

__global__ __launch_bounds__(kBlock) void k_seg_cells_clear(const sg_seg_sys* __restrict__ sys,
                                                            const int64_t* __restrict__ pfx,
                                                            int nsys) {
    int64_t lb;
    const int k = sg_seg_find(pfx, nsys, blockIdx.x, &lb);
    const sg_seg_sys& S = sys[k];
    cells_clear_block(S.g, S.count, S.hmax, lb, pfx[k + 1] - pfx[k]);
}

__global__ __launch_bounds__(kBlock) void k_seg_keys_count(const sg_seg_sys* __restrict__ sys,
                                                           const int64_t* __restrict__ pfx,
                                                           int nsys) {
    int64_t lb;
    const sg_seg_sys& S = sys[sg_seg_find(pfx, nsys, blockIdx.x, &lb)];
    if (S.g->err & SGE_SORT_FATAL) return;
    const int64_t i = lb * kBlock + threadIdx.x;
    keys_count_wave(S.x, S.y, S.z, S.h, S.m, i, i < S.ng, S.g, S.key, S.count, S.hmax,
                    reinterpret_cast<sg_prec*>(S.sph.f64));
}

// which = 0: cell counts -> cell offsets (n = M from the grid, bounded by
// the cell capacity); 1: neighbour counts -> CSR offsets (n = N_g)
__device__ inline void seg_scan_args(const sg_seg_sys& S, int which, const int32_t** in,
                                     int64_t** out, int64_t* n) {
    if (which == 0) {
        *in = S.count;
        *out = S.off;
        *n = S.g->M < S.cell_cap ? S.g->M : S.cell_cap;
    } else {
        *in = S.ncnt;
        *out = const_cast<int64_t*>(S.sph.nbr_off);
        *n = S.ng;
    }
}

__global__ __launch_bounds__(kBlock) void k_seg_scan_reduce(const sg_seg_sys* __restrict__ sys,
                                                            const int64_t* __restrict__ pfx,
                                                            int nsys, int which) {
    int64_t tile;
    const sg_seg_sys& S = sys[sg_seg_find(pfx, nsys, blockIdx.x, &tile)];
    const int32_t* in;
    int64_t* out;
    int64_t n;
    seg_scan_args(S, which, &in, &out, &n);
    scan_reduce_tile(in, n, tile, (int64_t*)S.scan);
}

__global__ __launch_bounds__(256) void k_seg_scan_bsums(const sg_seg_sys* __restrict__ sys,
                                                        int which) {
    const sg_seg_sys& S = sys[blockIdx.x];
    if (S.ng == 0) return;
    const int32_t* in;
    int64_t* out;
    int64_t n;
    seg_scan_args(S, which, &in, &out, &n);
    scan_bsums_block((int64_t*)S.scan, n, out);
}

__global__ __launch_bounds__(kBlock) void k_seg_scan_down(const sg_seg_sys* __restrict__ sys,
                                                          const int64_t* __restrict__ pfx,
                                                          int nsys, int which) {
    int64_t tile;
    const sg_seg_sys& S = sys[sg_seg_find(pfx, nsys, blockIdx.x, &tile)];
    const int32_t* in;
    int64_t* out;
    int64_t n;
    seg_scan_args(S, which, &in, &out, &n);
    scan_down_tile(in, out, n, tile, ((const int64_t*)S.scan)[tile]);
}

// Cell-key radix pass `pass` of every system (the per-system buffers'
// ping-pong of sg_launch_gas_order); the last pass writes the order.
__device__ inline void seg_gas_bufs(const sg_seg_sys& S, int pass, const uint32_t** kin,
                                    const int32_t** vin) {
    *kin = pass == 0 ? (const uint32_t*)S.key : (((pass - 1) & 1) ? S.gk1 : S.gk0);
    *vin = pass == 0 ? nullptr : (((pass - 1) & 1) ? S.gv1 : S.gv0);
}

__global__ __launch_bounds__(kBlock) void k_seg_gas_hist(const sg_seg_sys* __restrict__ sys,
                                                         const int64_t* __restrict__ pfx,
                                                         int nsys, int pass) {
    int64_t tile;
    const sg_seg_sys& S = sys[sg_seg_find(pfx, nsys, blockIdx.x, &tile)];
    const uint32_t* kin;
    const int32_t* vin;
    seg_gas_bufs(S, pass, &kin, &vin);
    radix_hist_tile(kin, S.ng, kRadixBits * pass, S.gntiles, S.ghist, tile);
}

__global__ __launch_bounds__(kBlock) void k_seg_gas_scatter(const sg_seg_sys* __restrict__ sys,
                                                            const int64_t* __restrict__ pfx,
                                                            int nsys, int pass, int last) {
    int64_t tile;
    const sg_seg_sys& S = sys[sg_seg_find(pfx, nsys, blockIdx.x, &tile)];
    const uint32_t* kin;
    const int32_t* vin;
    seg_gas_bufs(S, pass, &kin, &vin);
    int32_t* vout = last ? const_cast<int32_t*>(S.sph.perm) : ((pass & 1) ? S.gv1 : S.gv0);
    radix_scatter_tile(kin, vin, S.ng, kRadixBits * pass, S.gntiles, S.goffs,
                       (pass & 1) ? S.gk1 : S.gk0, vout, tile);
}

__global__ __launch_bounds__(kBlock) void k_seg_gather_gas(const sg_seg_sys* __restrict__ sys,
                                                           const int64_t* __restrict__ pfx,
                                                           int nsys) {
    int64_t lb;
    const sg_seg_sys& S = sys[sg_seg_find(pfx, nsys, blockIdx.x, &lb)];
    if (S.g->err & SGE_SORT_FATAL) return;
    const int64_t s = lb * kBlock + threadIdx.x;
    const sg_sph_bufs& b = S.sph;
    gather_one(b.perm, s, S.ng, reinterpret_cast<const sg_prec*>(b.f64), b.xs, b.ys, b.zs, b.hs,
               b.ms, b.prec, true);
}

inline unsigned grid_for(int64_t n, int per_block) {
    int64_t b = (n + per_block - 1) / per_block;
    return (unsigned)(b < 1 ? 1 : b);
}

}  // namespace

// ----------------------------------------------------------- launchers --

size_t sg_scan_tmp_bytes(int64_t cap) {
    return sizeof(int64_t) * (size_t)((cap + kScanTile - 1) / kScanTile + 1);
}

// Both ways: three launches of 4.5-5 us each and an idle chip in the middle
// one, against two; the sums of 1024 tiles (2097152 entries) cost a workgroup
// less than a launch.
void sg_launch_scan(const int32_t* in, int64_t* out, int64_t n_host, const int64_t* n_dev,
                    int64_t cap, void* tmp, hipStream_t st, sg_grid_dev* chk, int64_t nnz_cap) {
    const unsigned nb = grid_for(cap, kScanTile);
    int64_t* bsum = (int64_t*)tmp;
    hipLaunchKernelGGL(k_scan_reduce, dim3(nb), dim3(kBlock), 0, st, in, n_host, n_dev, cap, bsum);
    if (nb <= kScanOwn) {
        hipLaunchKernelGGL(k_scan_down_own, dim3(nb), dim3(kBlock), 0, st, in, out, n_host, n_dev,
                           cap, bsum, chk, nnz_cap);
        return;
    }
    hipLaunchKernelGGL(k_scan_bsums, dim3(1), dim3(256), 0, st, bsum, n_host, n_dev, cap, out);
    hipLaunchKernelGGL(k_scan_down, dim3(nb), dim3(kBlock), 0, st, in, out, n_host, n_dev, cap,
                       bsum);
    if (chk) hipLaunchKernelGGL(k_nbr_check, dim3(1), dim3(64), 0, st, chk, out, n_host, nnz_cap);
}

void sg_launch_status_clear(sg_grid_dev* g, bool record, hipStream_t st) {
    hipLaunchKernelGGL(k_status_clear, dim3(1), dim3(64), 0, st, g, record ? 1 : 0);
}

// Whole cell tables of up to this many cells are cleared beside the level
// bounds (12 bytes a cell, a few us at most) instead of by a launch of their own.
constexpr int64_t kClearWhole = 1 << 20;

// The one-workgroup kernels take up to kSmall keys, and the gas takes them by
// the number of all particles: beside a gravity kernel that fills the compute
// units a workgroup of 1024 lanes waits for its end.
bool sg_gas_small(int64_t n, int64_t cell_cap) {
    return n <= kSmall && cell_cap <= kClearWhole;
}

void sg_launch_gas_small(const double* x, const double* y, const double* z, const double* h,
                         const double* m, int64_t ng, sg_grid_dev* g, int64_t cell_cap,
                         int32_t* key, void* tmp, int32_t* perm, double* xs, double* ys, double* zs,
                         double* hs, double* ms, sg_prec* prec, int precision, int64_t* off,
                         int32_t* count, unsigned long long* hmax, hipStream_t st) {
    uint32_t* const sorted = static_cast<uint32_t*>(tmp);
    hipLaunchKernelGGL(k_keys_small, dim3(1), dim3(kSmallBlock), 0, st, x, y, z, h, (int)ng, g,
                       sg_gas_radix_passes(cell_cap), key, sorted, perm);
    const unsigned nbg = grid_for(ng, kBlock);
    unsigned nbc = grid_for(cell_cap + 1, kBlock);
    if (nbc > 2048) nbc = 2048;
    hipLaunchKernelGGL(k_gather_gas_small, dim3(nbg + nbc), dim3(kBlock), 0, st, perm, ng, g, x, y,
                       z, h, m, xs, ys, zs, hs, ms, prec, precision == SG_FP32C ? 1 : 0, (int)nbg,
                       sorted, off, count, hmax);
}

// Workgroups of k_grid_levels: each ends with eight device atomics a level on
// the same few lines, one after the other.  Sort stage in us with at most
// 1024 / 256 / 128 / 64 of them: 65536 particles 66 / 66 / 60 / 57; 131071 114
// / 99 / 93 / 90; 262144 170 / 128 / 123 / 123; 1048576 286 / 249 / 253 / 272.
static unsigned grid_blocks(int64_t ng) {
    const unsigned few = grid_for(ng, kBlock), many = grid_for(ng, 16 * kBlock);
    const unsigned lo = few < 64 ? few : 64, hi = many < 256 ? many : 256;
    return lo > hi ? lo : hi;
}

void sg_launch_grid(const double* x, const double* y, const double* z, const double* h, int64_t ng,
                    sg_grid_dev* g, int32_t* count, unsigned long long* hmax, int64_t cell_cap,
                    int cell_scale_log2, hipStream_t st) {
    const unsigned nb = grid_blocks(ng);
    const bool whole = cell_cap <= kClearWhole;
    unsigned ncl = whole ? grid_for(cell_cap, 4 * kBlock) : 0;
    if (ncl > 512) ncl = 512;
    const double scale = cell_scale_log2 < 0 ? 0.5 : (cell_scale_log2 > 0 ? 2.0 : 1.0);
    hipLaunchKernelGGL(k_grid_levels, dim3(nb + ncl), dim3(kBlock), 0, st, x, y, z, h, ng, g,
                       cell_cap, scale, count, hmax, cell_cap, nb);
    if (whole) return;
    unsigned nc = grid_for(cell_cap, kBlock);
    if (nc > 4096) nc = 4096;
    hipLaunchKernelGGL(k_cells_clear, dim3(nc), dim3(kBlock), 0, st, g, count, hmax);
}

void sg_launch_gas_keys(const double* x, const double* y, const double* z, const double* h,
                        const double* m, int64_t ng, sg_grid_dev* g, int32_t* key, sg_prec* pin,
                        hipStream_t st) {
    hipLaunchKernelGGL(k_gas_keys, dim3(grid_for(ng, kBlock)), dim3(kBlock), 0, st, x, y, z, h, m,
                       ng, g, key, pin);
}

void sg_launch_gather_gas(const int32_t* perm, int64_t ng, const sg_grid_dev* g,
                          const sg_prec* pin, double* xs, double* ys, double* zs, double* hs,
                          double* ms, sg_prec* prec, int precision, const uint32_t* keys,
                          int32_t* count, unsigned long long* hmax, hipStream_t st) {
    hipLaunchKernelGGL(k_gather_gas, dim3(grid_for(ng, kBlock)), dim3(kBlock), 0, st, perm, ng,
                       g, pin, xs, ys, zs, hs, ms, prec, precision == SG_FP32C ? 1 : 0, keys, count,
                       hmax);
}

// Bisection costs log2(N_g) dependent reads a cell, the scan three launches.
bool sg_offsets_by_bisection(int64_t ng, int64_t cell_cap) {
    return ng <= 65536 && cell_cap <= kClearWhole;
}

void sg_launch_gather_gas_off(const int32_t* perm, int64_t ng, const sg_grid_dev* g,
                              const sg_prec* pin, double* xs, double* ys, double* zs, double* hs,
                              double* ms, sg_prec* prec, int precision, const uint32_t* keys,
                              int64_t* off, int64_t cell_cap, int32_t* count,
                              unsigned long long* hmax, hipStream_t st) {
    const unsigned nbg = grid_for(ng, kBlock);
    unsigned nbc = grid_for(cell_cap + 1, kBlock);
    if (nbc > 2048) nbc = 2048;
    hipLaunchKernelGGL(k_gather_gas_off, dim3(nbg + nbc), dim3(kBlock), 0, st, perm, ng, g, pin,
                       xs, ys, zs, hs, ms, prec, precision == SG_FP32C ? 1 : 0, (int)nbg, keys, off,
                       count, hmax);
}

// Workspace of the Morton order: two key/value buffers, the digit histogram
// and its offsets, and the scan scratch.
static void morton_layout(int64_t n, size_t* o_k1, size_t* o_v0, size_t* o_v1, size_t* o_hist,
                          size_t* o_offs, size_t* o_scan, size_t* total) {
    auto al = [](size_t v) { return (v + 255) & ~(size_t)255; };
    const int64_t ntiles = (n + kRadixTile - 1) / kRadixTile;
    const int64_t nh = kBuckets * (ntiles > 0 ? ntiles : 1);
    size_t o = 0;
    o += al(sizeof(uint32_t) * (size_t)n);  // k0 at 0
    *o_k1 = o;
    o += al(sizeof(uint32_t) * (size_t)n);
    *o_v0 = o;
    o += al(sizeof(int32_t) * (size_t)n);
    *o_v1 = o;
    o += al(sizeof(int32_t) * (size_t)n);
    *o_hist = o;
    o += al(sizeof(int32_t) * (size_t)nh);
    *o_offs = o;
    o += al(sizeof(int64_t) * (size_t)(nh + 1));
    *o_scan = o;
    o += al(sg_scan_tmp_bytes(nh));
    *total = o;
}

size_t sg_morton_tmp_bytes(int64_t n) {
    size_t a, b, c, d, e, f, t;
    morton_layout(n, &a, &b, &c, &d, &e, &f, &t);
    return t;
}

int64_t sg_radix_tiles(int64_t n) { return (n + kRadixTile - 1) / kRadixTile; }
int64_t sg_scan_tiles(int64_t cap) { return grid_for(cap, kScanTile); }
int64_t sg_cells_clear_blocks(int64_t cell_cap) {
    const int64_t nb = grid_for(cell_cap, kBlock);
    return nb > 256 ? 256 : nb;
}

static void seg_scan(const sg_seg& s, int which, hipStream_t st) {
    const int q = which == 0 ? SG_SEG_SCAN_C : SG_SEG_SCAN_G;
    const int64_t* p = s.pfx + q * (s.nsys + 1);
    if (s.nblk[q] == 0) return;
    hipLaunchKernelGGL(k_seg_scan_reduce, dim3((unsigned)s.nblk[q]), dim3(kBlock), 0, st, s.sys, p,
                       s.nsys, which);
    hipLaunchKernelGGL(k_seg_scan_bsums, dim3((unsigned)s.nsys), dim3(256), 0, st, s.sys, which);
    hipLaunchKernelGGL(k_seg_scan_down, dim3((unsigned)s.nblk[q]), dim3(kBlock), 0, st, s.sys, p,
                       s.nsys, which);
}

void sg_seg_launch_sort(const sg_seg& s, hipStream_t st) {
    if (s.nblk[SG_SEG_NG] == 0) return;
    const int64_t* png = s.pfx + SG_SEG_NG * (s.nsys + 1);
    const int64_t* pcl = s.pfx + SG_SEG_CELLS * (s.nsys + 1);
    const unsigned nbg = (unsigned)s.nblk[SG_SEG_NG];
    hipLaunchKernelGGL(k_seg_grid_levels, dim3(nbg), dim3(kBlock), 0, st, s.sys, png, s.nsys);
    hipLaunchKernelGGL(k_seg_grid_finish, dim3((unsigned)s.nsys), dim3(64), 0, st, s.sys);
    hipLaunchKernelGGL(k_seg_cells_clear, dim3((unsigned)s.nblk[SG_SEG_CELLS]), dim3(kBlock), 0, st,
                       s.sys, pcl, s.nsys);
    hipLaunchKernelGGL(k_seg_keys_count, dim3(nbg), dim3(kBlock), 0, st, s.sys, png, s.nsys);
    seg_scan(s, 0, st);
    const int64_t* pgt = s.pfx + SG_SEG_GTILES * (s.nsys + 1);
    for (int pass = 0; pass < s.gas_passes; ++pass) {
        hipLaunchKernelGGL(k_seg_gas_hist, dim3((unsigned)s.nblk[SG_SEG_GTILES]), dim3(kBlock), 0,
                           st, s.sys, pgt, s.nsys, pass);
        hipLaunchKernelGGL(k_seg_scan_hist, dim3((unsigned)s.nsys), dim3(kSegScanBlock), 0, st,
                           s.sys, 1);
        hipLaunchKernelGGL(k_seg_gas_scatter, dim3((unsigned)s.nblk[SG_SEG_GTILES]), dim3(kBlock),
                           0, st, s.sys, pgt, s.nsys, pass, pass == s.gas_passes - 1 ? 1 : 0);
    }
    hipLaunchKernelGGL(k_seg_gather_gas, dim3(nbg), dim3(kBlock), 0, st, s.sys, png, s.nsys);
}

void sg_seg_launch_scan_nbr(const sg_seg& s, hipStream_t st) { seg_scan(s, 1, st); }

void sg_morton_ptrs(void* tmp, int64_t n, uint32_t** k0, uint32_t** k1, int32_t** v0,
                    int32_t** v1, int32_t** hist, int64_t** offs, int64_t* ntiles) {
    size_t o_k1, o_v0, o_v1, o_hist, o_offs, o_scan, total;
    morton_layout(n, &o_k1, &o_v0, &o_v1, &o_hist, &o_offs, &o_scan, &total);
    char* base = (char*)tmp;
    *k0 = (uint32_t*)base;
    *k1 = (uint32_t*)(base + o_k1);
    *v0 = (int32_t*)(base + o_v0);
    *v1 = (int32_t*)(base + o_v1);
    *hist = (int32_t*)(base + o_hist);
    *offs = (int64_t*)(base + o_offs);
    *ntiles = sg_radix_tiles(n);
}

void sg_seg_launch_morton_order(const sg_seg& s, hipStream_t st) {
    const int64_t* pn = s.pfx + SG_SEG_N * (s.nsys + 1);
    const int64_t* pt = s.pfx + SG_SEG_TILES * (s.nsys + 1);
    if (s.nblk[SG_SEG_N] == 0) return;
    hipLaunchKernelGGL(k_seg_gbox, dim3((unsigned)s.nblk[SG_SEG_N]), dim3(kBlock), 0, st, s.sys, pn,
                       s.nsys);
    hipLaunchKernelGGL(k_seg_morton_keys, dim3((unsigned)s.nblk[SG_SEG_N]), dim3(kBlock), 0, st,
                       s.sys, pn, s.nsys);
    for (int pass = 0; pass < kRadixPasses; ++pass) {
        hipLaunchKernelGGL(k_seg_radix_hist, dim3((unsigned)s.nblk[SG_SEG_TILES]), dim3(kBlock), 0,
                           st, s.sys, pt, s.nsys, pass);
        hipLaunchKernelGGL(k_seg_scan_hist, dim3((unsigned)s.nsys), dim3(kSegScanBlock), 0, st,
                           s.sys, 0);
        hipLaunchKernelGGL(k_seg_radix_scatter, dim3((unsigned)s.nblk[SG_SEG_TILES]), dim3(kBlock),
                           0, st, s.sys, pt, s.nsys, pass);
    }
}

int sg_gas_radix_passes(int64_t cell_cap) {
    uint64_t top = cell_cap > 1 ? (uint64_t)(cell_cap - 1) : 1u;   // largest key
    int bits = 0;
    while (top) {
        ++bits;
        top >>= 1;
    }
    return (bits + kRadixBits - 1) / kRadixBits;
}

// One stable pass over digit `shift` of n keys: two launches with rows of
// histograms where kRowTiles tiles do (smaller tiles where the histogram
// scratch, three rows for every 4096 keys, has room for their rows), else
// histogram, scan and scatter.
static void radix_pass(const uint32_t* kin, const int32_t* vin, int64_t n, int shift,
                       int32_t* hist, int64_t* offs, void* scan_tmp, uint32_t* kout, int32_t* vout,
                       hipStream_t st) {
    auto rows = [&](auto items) {
        constexpr int kItems = decltype(items)::value;
        const unsigned nt = grid_for(n, kBlock * kItems);
        hipLaunchKernelGGL((k_radix_hist_rows<kItems>), dim3(nt), dim3(kBlock), 0, st, kin, n,
                           shift, hist);
        hipLaunchKernelGGL((k_radix_scatter_rows<kItems>), dim3(nt), dim3(kBlock), 0, st, kin, vin,
                           n, shift, (int)nt, hist, kout, vout);
    };
    if (n <= 3 * kBlock * 4) return rows(std::integral_constant<int, 4>());
    if (n <= kRowTiles * kBlock * 8) return rows(std::integral_constant<int, 8>());
    if (n <= kRowTiles * kBlock * 16) return rows(std::integral_constant<int, 16>());
    const int64_t ntiles = sg_radix_tiles(n);
    hipLaunchKernelGGL(k_radix_hist, dim3((unsigned)ntiles), dim3(kBlock), 0, st, kin, n, shift,
                       ntiles, hist);
    sg_launch_scan(hist, offs, kBuckets * ntiles, nullptr, kBuckets * ntiles, scan_tmp, st);
    hipLaunchKernelGGL(k_radix_scatter, dim3((unsigned)ntiles), dim3(kBlock), 0, st, kin, vin, n,
                       shift, ntiles, offs, kout, vout);
}

const uint32_t* sg_launch_gas_order(const int32_t* key, int64_t ng, int64_t cell_cap, void* tmp,
                                    int32_t* perm, hipStream_t st) {
    uint32_t *k0, *k1;
    int32_t *v0, *v1, *hist;
    int64_t* offs;
    int64_t ntiles;
    sg_morton_ptrs(tmp, ng, &k0, &k1, &v0, &v1, &hist, &offs, &ntiles);
    size_t o_k1, o_v0, o_v1, o_hist, o_offs, o_scan, total;
    morton_layout(ng, &o_k1, &o_v0, &o_v1, &o_hist, &o_offs, &o_scan, &total);
    void* scan_tmp = (char*)tmp + o_scan;
    uint32_t* kb[2] = {k0, k1};
    int32_t* vb[2] = {v0, v1};
    const int passes = sg_gas_radix_passes(cell_cap);
    const uint32_t* kin = (const uint32_t*)key;        // keys are >= 0
    const int32_t* vin = nullptr;                        // ids 0 .. ng-1
    for (int pass = 0; pass < passes; ++pass) {
        int32_t* vout = pass == passes - 1 ? perm : vb[pass & 1];
        radix_pass(kin, vin, ng, kRadixBits * pass, hist, offs, scan_tmp, kb[pass & 1], vout, st);
        kin = kb[pass & 1];
        vin = vb[pass & 1];
    }
    return kin;
}

void sg_launch_morton_order(const double* x, const double* y, const double* z, int64_t n,
                            sg_grid_dev* g, int32_t* order, void* tmp, hipStream_t st) {
    size_t o_k1, o_v0, o_v1, o_hist, o_offs, o_scan, total;
    morton_layout(n, &o_k1, &o_v0, &o_v1, &o_hist, &o_offs, &o_scan, &total);
    char* base = (char*)tmp;
    uint32_t* k[2] = {(uint32_t*)base, (uint32_t*)(base + o_k1)};
    int32_t* v[2] = {(int32_t*)(base + o_v0), (int32_t*)(base + o_v1)};
    int32_t* hist = (int32_t*)(base + o_hist);
    int64_t* offs = (int64_t*)(base + o_offs);
    void* scan_tmp = base + o_scan;
    unsigned nb = grid_for(n, kBlock);
    if (n <= kSmall) {
        hipLaunchKernelGGL(k_morton_small, dim3(1), dim3(kSmallBlock), 0, st, x, y, z, (int)n, g,
                           order);
        return;
    }
    hipLaunchKernelGGL(k_gbox, dim3(nb > 512 ? 512 : nb), dim3(kBlock), 0, st, x, y, z, n, g);
    hipLaunchKernelGGL(k_morton_keys, dim3(nb), dim3(kBlock), 0, st, x, y, z, n, g, k[0]);
    // the first pass takes the values 0 .. n-1 from the element indices
    int cur = 0;
    for (int pass = 0; pass < kRadixPasses; ++pass) {
        int32_t* vo = (pass == kRadixPasses - 1) ? order : v[cur ^ 1];
        radix_pass(k[cur], pass == 0 ? nullptr : v[cur], n, kRadixBits * pass, hist, offs, scan_tmp,
                   k[cur ^ 1], vo, st);
        cur ^= 1;
    }
}
