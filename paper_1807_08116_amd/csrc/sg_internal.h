// sg_internal.h -- device-side structures and launcher declarations shared by
// the translation units of libsphgrav.so (not part of the public ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sphgrav.h"

#define SG_MAXLEV SG_MAX_LEVELS
#define SG_BINADES SG_MAXLEV

// Device error bits (latched; cleared by sg_create / sg_bind_state).
enum : uint32_t {
    SGE_LEVELS = 1u,      // smoothing lengths need more than SG_MAXLEV levels
    SGE_CELLS = 2u,       // M > cell_cap
    SGE_NNZ = 4u,         // neighbour pairs > nnz_cap
    SGE_NONFINITE = 8u,   // non-finite position, h <= 0 or non-finite h
    SGE_GRID = 16u,       // a level's cell count does not fit in int32
    SGE_GNONFINITE = 32u, // non-finite position met by the gravity preparation
                          // (apart from SGE_NONFINITE, which the neighbour
                          // build reads: the two chains may run concurrently)
};
#define SGE_SORT_FATAL (SGE_LEVELS | SGE_CELLS | SGE_NONFINITE | SGE_GRID)

// Workgroups of a launch are dealt to the 8 XCDs of the chip round-robin,
// and each XCD has its own L2.  Kernels whose neighbouring targets share
// data (neighbour gathers over slot-ordered particles) remap the block
// index so that each XCD walks one contiguous range of blocks: a bijection
// of [0, nb), whatever the hardware's actual placement.
constexpr int kXcds = 8;
__device__ inline int64_t xcd_block(int64_t b, int64_t nb) {
    const int64_t per = nb / kXcds, rem = nb % kXcds;
    const int64_t x = b % kXcds, k = b / kXcds;
    return x * per + (x < rem ? x : rem) + k;
}

// Chunked variant: chunks of G consecutive logical blocks are dealt to the
// XCDs in turn, so every XCD takes work from all parts of the range while
// the blocks of one chunk share an L2.  Blocks in the tail (the last
// nb mod 8G) keep their own index.  A bijection of [0, nb).
__device__ inline int64_t xcd_chunk_block(int64_t b, int64_t nb, int64_t G) {
    const int64_t span = kXcds * G;
    if (b >= nb / span * span) return b;
    const int64_t x = b % kXcds, k = b / kXcds;
    return ((k / G) * kXcds + x) * G + k % G;
}

// System of block b of a segmented launch: the largest s with p[s] <= b
// (p = per-system prefix of block counts, p[0] = 0; systems without blocks
// are never found); *local = b - p[s].
__device__ inline int sg_seg_find(const int64_t* __restrict__ p, int nsys, int64_t b,
                                  int64_t* local) {
    int lo = 0, hi = nsys - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (p[mid] <= b) lo = mid;
        else hi = mid - 1;
    }
    *local = b - p[lo];
    return lo;
}

// Between a wavefront's LDS accesses that meet across lanes: the hardware
// keeps their order, this makes the compiler keep it too (no instruction).
__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Records moved by groups of lanes.  A lane that reads or writes a record of
// its own touches a cache line of its own with every 16 bytes, and the vector
// memory's address unit takes them one line a cycle: gathers of 64-byte
// records kept it busy all the time (force pass at 1048576 gas particles).
// Here the four lanes of a quad move one record per instruction, 16 bytes a
// lane, so a quad's instruction touches one line, and a 4x4 transpose of
// 16-byte pieces gives every lane its own record; pairs of lanes move 32-byte
// records alike.  FP32C passes at that size: force 533 -> 340 us (the vector
// ALU is busy throughout now), density 285 -> 212.  All lanes of the quad
// must be active; bases are 64-byte (32-byte) aligned.
template <int kCtrl>
__device__ inline uint32_t dpp_quad(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kCtrl, 0xf, 0xf, true);
}
// the lower lane's b <-> the upper lane's a
template <int kCtrl>
__device__ inline void quad_swap(uint32_t& a, uint32_t& b, bool upper) {
    const uint32_t xa = dpp_quad<kCtrl>(a), xb = dpp_quad<kCtrl>(b);   // with all lanes active
    a = upper ? xb : a;
    b = upper ? b : xa;
}
template <int kCtrl>
__device__ inline void quad_swap(uint4& a, uint4& b, bool upper) {
    quad_swap<kCtrl>(a.x, b.x, upper);
    quad_swap<kCtrl>(a.y, b.y, upper);
    quad_swap<kCtrl>(a.z, b.z, upper);
    quad_swap<kCtrl>(a.w, b.w, upper);
}
// v[p] of lane r <-> v[r] of lane p
__device__ inline void quad_transpose(uint4 (&v)[4]) {
    const bool b0 = threadIdx.x & 1, b1 = threadIdx.x & 2;
    quad_swap<0xb1>(v[0], v[1], b0);
    quad_swap<0xb1>(v[2], v[3], b0);
    quad_swap<0x4e>(v[0], v[2], b1);
    quad_swap<0x4e>(v[1], v[3], b1);
}
// Record idx (64 bytes) of every lane.
__device__ inline void quad_load64(const void* base, int32_t idx, uint4 (&v)[4]) {
    const char* p = static_cast<const char*>(base) + 16 * (threadIdx.x & 3);
    const uint32_t i[4] = {dpp_quad<0x00>((uint32_t)idx), dpp_quad<0x55>((uint32_t)idx),
                           dpp_quad<0xaa>((uint32_t)idx), dpp_quad<0xff>((uint32_t)idx)};
    for (int k = 0; k < 4; ++k) v[k] = *reinterpret_cast<const uint4*>(p + 64 * (size_t)i[k]);
    quad_transpose(v);
}
// Record idx of every lane with idx >= 0.
__device__ inline void quad_store64(void* base, int32_t idx, uint4 (&v)[4]) {
    char* p = static_cast<char*>(base) + 16 * (threadIdx.x & 3);
    const int32_t i[4] = {(int32_t)dpp_quad<0x00>((uint32_t)idx), (int32_t)dpp_quad<0x55>((uint32_t)idx),
                          (int32_t)dpp_quad<0xaa>((uint32_t)idx), (int32_t)dpp_quad<0xff>((uint32_t)idx)};
    quad_transpose(v);
    for (int k = 0; k < 4; ++k)
        if (i[k] >= 0) *reinterpret_cast<uint4*>(p + 64 * (size_t)i[k]) = v[k];
}
__device__ inline void pair_load32(const void* base, int32_t idx, uint4 (&v)[2]) {
    const char* p = static_cast<const char*>(base) + 16 * (threadIdx.x & 1);
    const uint32_t i0 = dpp_quad<0xa0>((uint32_t)idx), i1 = dpp_quad<0xf5>((uint32_t)idx);
    v[0] = *reinterpret_cast<const uint4*>(p + 32 * (size_t)i0);
    v[1] = *reinterpret_cast<const uint4*>(p + 32 * (size_t)i1);
    quad_swap<0xb1>(v[0], v[1], threadIdx.x & 1);
}
__device__ inline void pair_store32(void* base, int32_t idx, uint4 (&v)[2]) {
    char* p = static_cast<char*>(base) + 16 * (threadIdx.x & 1);
    const int32_t i0 = (int32_t)dpp_quad<0xa0>((uint32_t)idx), i1 = (int32_t)dpp_quad<0xf5>((uint32_t)idx);
    quad_swap<0xb1>(v[0], v[1], threadIdx.x & 1);
    if (i0 >= 0) *reinterpret_cast<uint4*>(p + 32 * (size_t)i0) = v[0];
    if (i1 >= 0) *reinterpret_cast<uint4*>(p + 32 * (size_t)i1) = v[1];
}
// A record as its 16-byte pieces and back.
template <typename R, typename P, int K>
__device__ inline R rec_of(const P (&v)[K]) {
    static_assert(sizeof(R) == 16 * K, "whole record");
    R r;
    __builtin_memcpy(&r, &v, sizeof(R));
    return r;
}
template <typename R, int K>
__device__ inline void rec_to(const R& r, uint4 (&v)[K]) {
    static_assert(sizeof(R) == 16 * K, "whole record");
    __builtin_memcpy(&v, &r, sizeof(R));
}

// Grid of smoothing-length levels plus the device status word.  Lives in
// the workspace; written only by device code: the level fields by the
// neighbour build, the gravity-order box (glo, ghi) and the choice and scales
// of the pairwise gravity by the gravity preparation, the status word by both
// (atomic OR).
struct sg_grid_dev {
    // reduction inputs by binade of the cell side (its exponent modulo
    // SG_BINADES), as order-preserving u64 images of doubles
    struct binade {
        unsigned long long lo[3], hi[3], hmax, cnt;
    } bin[SG_BINADES];
    uint32_t emin, emax;               // smallest and largest exponent
    uint32_t ticket;                   // workgroups that have ended their part
    int32_t nlev;                      // (finished grid)
    // gravity preparation: whether the symmetric kernel may run (else the
    // one-sided one), and the scales (powers of two) of its fixed-point sums
    int32_t grav_sym;
    uint32_t err;                      // status
    double grav_S, grav_Sp;
    // finished grid (the cell side of level l is 1 / invL[l])
    double L0;
    double invL[SG_MAXLEV];
    double org[SG_MAXLEV][3];
    int64_t dim[SG_MAXLEV][3];
    int64_t base[SG_MAXLEV];
    int64_t ncell[SG_MAXLEV];
    unsigned long long npart[SG_MAXLEV];
    double hmaxlev[SG_MAXLEV];
    int64_t M;
    // gravity-order bounding box over all N (order-preserving u64 images)
    unsigned long long glo[3], ghi[3];
    // status
    int64_t need_cells, need_nnz;
    int64_t nnz;
};

// The number of list entries, against the capacity.
__device__ inline void nbr_check_total(sg_grid_dev* g, int64_t nnz, int64_t nnz_cap) {
    if (g->err & SGE_SORT_FATAL) {
        g->nnz = 0;
        return;
    }
    g->nnz = nnz;
    if (nnz > nnz_cap) {
        atomicOr(&g->err, SGE_NNZ);
        g->need_nnz = nnz;
    }
}

// Order-preserving map of doubles onto u64 (for integer atomic min/max).
__host__ __device__ inline unsigned long long sg_ord(double v) {
    unsigned long long b = (unsigned long long)__builtin_bit_cast(long long, v);
    return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}
__host__ __device__ inline double sg_unord(unsigned long long m) {
    unsigned long long b = (m >> 63) ? (m & 0x7fffffffffffffffull) : ~m;
    return __builtin_bit_cast(double, (long long)b);
}

// ---- launchers (each defined in the translation unit of its kernels) ----
// Scans: exclusive prefix sums of int32 counts into int64 offsets, with
// out[n] = total.  n is read from *n_dev when n_dev != nullptr (device-side
// sizes), else n_host; cap bounds the launch.  chk: in holds the numbers of
// neighbours; their total becomes chk->nnz and is checked against nnz_cap.
size_t sg_scan_tmp_bytes(int64_t cap);
void sg_launch_scan(const int32_t* in, int64_t* out, int64_t n_host, const int64_t* n_dev,
                    int64_t cap, void* tmp, hipStream_t st,
                    sg_grid_dev* chk = nullptr, int64_t nnz_cap = 0);

// Gas sort chain.
// Clear the error word; record: also the grid record and the reduction
// inputs (a newly bound state).
void sg_launch_status_clear(sg_grid_dev* g, bool record, hipStream_t st);
// Grid rule (minimum h, level bounds, cell sides and offsets) and cleared
// cell counts and maxima.
void sg_launch_grid(const double* x, const double* y, const double* z, const double* h, int64_t ng,
                    sg_grid_dev* g, int32_t* count, unsigned long long* hmax, int64_t cell_cap,
                    int cell_scale_log2, hipStream_t st);
// Cell keys; also each particle's record (x, y, z, h, m) in particle order
// into pin [ng] (scratch the gather reads).
struct sg_prec;
void sg_launch_gas_keys(const double* x, const double* y, const double* z, const double* h,
                        const double* m, int64_t ng, sg_grid_dev* g, int32_t* key, sg_prec* pin,
                        hipStream_t st);
// Stable order of the gas by cell key (ascending id inside a cell): LSD
// radix sort of the keys with 10-bit digits, enough passes for keys below
// cell_cap; tmp: sg_morton_tmp_bytes(ng) bytes.
int sg_gas_radix_passes(int64_t cell_cap);
// Returns the keys in sorted order (in tmp).
const uint32_t* sg_launch_gas_order(const int32_t* key, int64_t ng, int64_t cell_cap, void* tmp,
                         int32_t* perm, hipStream_t st);
// Keys, order, gather, cell offsets, counts and maxima in two launches, for
// sizes where sg_gas_small says so; n: all particles.
struct sg_prec;
bool sg_gas_small(int64_t n, int64_t cell_cap);
void sg_launch_gas_small(const double* x, const double* y, const double* z, const double* h,
                         const double* m, int64_t ng, sg_grid_dev* g, int64_t cell_cap,
                         int32_t* key, void* tmp, int32_t* perm, double* xs, double* ys, double* zs,
                         double* hs, double* ms, sg_prec* prec, int precision, int64_t* off,
                         int32_t* count, unsigned long long* hmax, hipStream_t st);
void sg_launch_gather_gas(const int32_t* perm, int64_t ng, const sg_grid_dev* g,
                          const sg_prec* pin, double* xs, double* ys, double* zs, double* hs,
                          double* ms, sg_prec* prec, int precision, const uint32_t* keys,
                          int32_t* count, unsigned long long* hmax, hipStream_t st);
// The gather with the cell offsets from the sorted keys beside it, for sizes
// where that beats the scan of the counts.
bool sg_offsets_by_bisection(int64_t ng, int64_t cell_cap);
void sg_launch_gather_gas_off(const int32_t* perm, int64_t ng, const sg_grid_dev* g,
                              const sg_prec* pin, double* xs, double* ys, double* zs, double* hs,
                              double* ms, sg_prec* prec, int precision, const uint32_t* keys,
                              int64_t* off, int64_t cell_cap, int32_t* count, unsigned long long* hmax,
                              hipStream_t st);

// Neighbour lists.
// Neighbour search: per-target slots of fixed length (sg_nbr_slot_bytes),
// counts, then (after the scan and the capacity check) the copy into CSR.
size_t sg_nbr_slot_bytes(int64_t ng);
void sg_launch_nbr_search(const sg_grid_dev* g, int64_t ng, const double* xs, const double* ys,
                          const double* zs, const double* hs, const int64_t* off,
                          const int32_t* perm, const int32_t* key, int32_t* cnt, int32_t* slots,
                          hipStream_t st);
// CSR offsets from the counts, the capacity check and the copy into the rows
// (scan: scratch of sg_scan_tmp_bytes(ng)).
void sg_launch_nbr_finish(sg_grid_dev* g, int64_t ng, const double* xs, const double* ys,
                          const double* zs, const double* hs, const int64_t* off,
                          const int32_t* cnt, const int32_t* slots, int64_t nnz_cap, void* scan,
                          int64_t* nbr_off, int32_t* nbr_idx, hipStream_t st);

// SPH.  Per-particle data in sorted-slot order is packed into one record
// per particle, so a neighbour gather touches one or two cache lines.
struct alignas(64) sg_prec {          // positions for the FP64 density pass
    double x, y, z, h, m, pad[3];
};
struct alignas(32) sg_prec32 {        // the same for the FP32C form
    double x, y, z;
    float h, m;
};
// FP64 force pass, in two arrays: a particle's 64 bytes, then (after all of
// them) its 32 bytes (P = p / rho^2).
struct alignas(64) sg_frec64 {
    double x, y, z, h, m, vx, vy, vz;
};
struct alignas(32) sg_frec64b {
    double rho, P, c, pad;
};
struct alignas(64) sg_frec32 {        // FP32C force pass (FP64 positions)
    double x, y, z;
    float h, m, vx, vy, vz, rho, P, c, pad[2];
};
struct sg_sph_bufs {
    double *xs, *ys, *zs, *hs, *ms;     // sorted SoA (neighbour search, h update)
    double* rho_s;                      // density by slot
    sg_prec* prec;                      // sg_prec, or (FP32C) sg_prec32 records
    sg_frec64* f64;
    sg_frec64b* f64b;
    sg_frec32* f32;
    const int32_t* perm;
    const int64_t* nbr_off;
    const int32_t* nbr_idx;
    // (vx, vy, vz, e) of each gas particle in particle order, 32 bytes each,
    // packed for the record build's random reads; it borrows the
    // neighbour-search slots, which are free once the lists are copied
    double* ve;
};
void sg_launch_density(const sg_sph_bufs& b, const sg_grid_dev* g, int64_t ng, int precision,
                       double* rho_out, hipStream_t st);
// precision: SG_FP64 or SG_FP32C, or kPrepCfl for the time-step rule's records
// (those of the FP64 pass with the sound speed as their mass, no second part).
constexpr int kPrepCfl = 2;
void sg_launch_sph_prep(const sg_sph_bufs& b, const sg_grid_dev* g, int64_t ng, int precision,
                        double gamma, const double* vx, const double* vy, const double* vz,
                        const double* e, hipStream_t st);
// SPH acceleration (asx/asy/asz) and de/dt, both in particle order.
void sg_launch_sph_force(const sg_sph_bufs& b, const sg_grid_dev* g, int64_t ng, int precision,
                         double alpha, double beta, double eta, double* asx, double* asy,
                         double* asz, double* dedt, hipStream_t st);

// Step control: CFL time step into *out (device double) and h update.
void sg_launch_cfl(const sg_sph_bufs& b, const sg_grid_dev* g, int64_t ng, double alpha,
                   double beta, double eta, double C, const double* qx, const double* qy,
                   const double* qz, const double* dedt, double* out, hipStream_t st);
void sg_launch_update_h(const sg_sph_bufs& b, const sg_grid_dev* g, int64_t ng, double sigma,
                        double* h, hipStream_t st);

// Gravity.
struct sg_grav_args {
    const double *x, *y, *z, *m;
    int64_t n;
    double G, eps;
    int precision, ipl, split, with_pot;
    int tile;                           // sources per LDS tile: 128, 256 or 512
    int variant;                        // resolved: FP64 1/2 = difference form with FP32-/FP64-
                                        // seeded rsqrt, 3/4 = expanded far field (Morton order,
                                        // same seeds); FP32C 1 (the only one)
    const int32_t* order;               // FP32C, FP64 3/4: Morton order of the particles
    void* sorted;                       // FP32C, FP64 3/4: scratch of sg_grav_sorted_bytes(n)
    const double *xs, *ys, *zs, *ms;    // (set by the launcher) sorted copies
    const void* sbox;                   // (set by the launcher) sub-tile boxes
    double *gx, *gy, *gz, *gpot;        // outputs [n], particle order
    double* part;                       // split partials [4][split][n] when split > 1; the
                                        // symmetric kernel's fixed-point sums (sg_grav_sym_bytes)
    int sym;                            // symmetric kernel: targets per lane (1, 2 or 4), 0 = the
                                        // one-sided kernel alone
    int64_t sym_chunk, sym_period;      // tiles per workgroup (a multiple of the period), tiles
                                        // per rounding of the target-side sums
    sg_grid_dev* g;                     // error word (non-finite positions), scales and choice
};
size_t sg_grav_sorted_bytes(int64_t n);
size_t sg_grav_sym_bytes(int64_t n);
// FP32C: Morton-ordered copies of x, y, z, m and the boxes of their
// 64-particle runs (needs a.order and a.sorted); a non-finite position
// sets SGE_GNONFINITE in a.g's error word, and the Morton box is reset for
// the next order.
// Both return -1 (and launch nothing) when a required pointer is missing.
int sg_launch_grav_sorted(const sg_grav_args& a, hipStream_t st);
int sg_launch_gravity(const sg_grav_args& a, hipStream_t st);

// Symmetric kernel: 256-source tiles of the longest block list (its own
// block, (nb - 1) / 2 others, one more for half of the blocks when their
// number nb is even), t targets per lane.
inline int64_t sg_sym_tiles(int64_t n, int t) {
    const int64_t B = 256 * (int64_t)t, nb = (n + B - 1) / B;
    return t * (1 + nb / 2);
}

// Ensembles: one persistent launch over (system, block of 256*ipl targets)
// tasks of several systems in the FP32C form.
struct sg_ens_sys {
    const double *xs, *ys, *zs, *ms;    // Morton-sorted copies
    const void* sbox;                   // 64-particle boxes
    const int32_t* order;
    int64_t n;
    double *gx, *gy, *gz, *gp;          // outputs, particle order
    sg_grid_dev* g;
    long long* acc;                     // the symmetric kernel's sums (sg_grav_sym_bytes)
    int32_t sym, sym_period;            // the symmetric kernel serves this system (where the
                                        // device's choice, g->grav_sym, allows it)
};
struct sg_ens_task {
    int32_t sys, blk;
};
struct sg_sym_task {
    int32_t sys, blk, t0, t1;           // tiles [t0, t1) of the block's source list
};
void sg_grav_sorted_ptrs(void* sorted, int64_t n, const double** xs, const double** ys,
                         const double** zs, const double** ms, const void** sbox);
// The symmetric launch over its tasks (it resets both task counters first:
// d_counter[0] belongs to the one-sided launch, which follows it and takes
// the systems that the symmetric kernel does not serve).
void sg_launch_grav_ensemble_sym(const sg_ens_sys* d_sys, const sg_sym_task* d_tasks,
                                 int32_t ntasks, int32_t* d_counter, int with_pot, double eps,
                                 int t, int nblocks, hipStream_t st);
int sg_grav_sym_blocks_per_cu(int t);
void sg_launch_grav_ensemble(const sg_ens_sys* d_sys, const sg_ens_task* d_tasks, int32_t ntasks,
                             int32_t* d_counter, int with_pot, double eps, double G, int ipl,
                             int tile, int nblocks, hipStream_t st);
// Workgroups of the ensemble kernel that fit on one CU at once (>= 1).
int sg_grav_ensemble_blocks_per_cu(int ipl, int tile, int with_pot);

// Spatial (Morton) order of all N particles for the FP32C gravity targets.
size_t sg_morton_tmp_bytes(int64_t n);
void sg_launch_morton_order(const double* x, const double* y, const double* z, int64_t n,
                            sg_grid_dev* g, int32_t* order, void* tmp, hipStream_t st);

// Segmented launches: one launch covers a stage for every system of an
// ensemble.  Each system's pointers sit in a device table; a launch's
// blocks are dealt to systems by a prefix of per-system block counts (the
// block of a system is found by a search over that prefix, uniform per
// workgroup).  Each kernel body is the one of the per-system kernel, so
// results are the same bit for bit.
struct sg_seg_sys {
    // caller's state
    double *x, *y, *z, *vx, *vy, *vz, *m, *e, *ax, *ay, *az, *dedt, *rho;
    // workspace: predictor values, SPH and gravity parts
    double *vtx, *vty, *vtz, *et;
    double *asx, *asy, *asz;
    double *gx, *gy, *gz, *gp;
    long long* acc;                  // as in sg_ens_sys
    int32_t sym, pad;
    sg_sph_bufs sph;
    sg_grid_dev* g;
    // Morton order: key/value ping-pong buffers, digit histograms and
    // their offsets, the order, sorted copies and 64-particle boxes
    uint32_t *mk0, *mk1;
    int32_t *mv0, *mv1;
    int32_t* mhist;
    int64_t* moffs;
    int32_t* order;
    double *xs, *ys, *zs, *ms;
    void* sbox;
    // gas sort and neighbour lists
    double* h;                       // caller's smoothing lengths
    int32_t *key, *count, *ncnt, *slots;
    // radix sort of the cell keys (as the Morton buffers, for N_g)
    uint32_t *gk0, *gk1;
    int32_t *gv0, *gv1;
    int32_t* ghist;
    int64_t* goffs;
    int64_t gntiles;
    unsigned long long* hmax;
    int64_t* off;
    void* scan;                      // scan scratch (block sums)
    int64_t n, ng, ntiles, cell_cap, nnz_cap;
    double cell_scale;
    double gamma, alpha, beta, eta;
};
// Block prefixes of a segmented launch, per system: blocks of 256
// particles, of 256 gas particles, radix tiles, cell-clearing blocks
// (grid-stride, at most 256 per system), scan tiles of the cell counts and
// of the neighbour counts, blocks of the list copy (sg_compact_blocks),
// radix tiles of the gas, blocks of the SPH density and force passes
// (sg_sph_blocks) and of the neighbour search (sg_nbr_blocks).
enum {
    SG_SEG_N = 0, SG_SEG_NG = 1, SG_SEG_TILES = 2, SG_SEG_CELLS = 3, SG_SEG_SCAN_C = 4,
    SG_SEG_SCAN_G = 5, SG_SEG_CPT = 6, SG_SEG_GTILES = 7, SG_SEG_SPH = 8, SG_SEG_NBR = 9,
    SG_SEG_NPFX = 10
};
struct sg_seg {
    const sg_seg_sys* sys;           // [nsys], device
    const int64_t* pfx;              // [SG_SEG_NPFX][nsys + 1] block prefixes, device
    int32_t nsys;
    int32_t sym;                     // some system is served by the symmetric gravity
    double eps;
    int32_t nbr_targets;             // targets per wavefront of the neighbour search
    int32_t gas_passes;              // radix passes of the cell keys (largest over systems)
    int64_t nblk[SG_SEG_NPFX];       // totals of the prefixes (host)
};
// Host helpers for building the table.
void sg_morton_ptrs(void* tmp, int64_t n, uint32_t** k0, uint32_t** k1, int32_t** v0,
                    int32_t** v1, int32_t** hist, int64_t** offs, int64_t* ntiles);
int64_t sg_radix_tiles(int64_t n);
int64_t sg_scan_tiles(int64_t cap);          // blocks of one sg_launch_scan pass
int64_t sg_cells_clear_blocks(int64_t cell_cap);
// Stages (each one launch, or a few, for all systems).
// (predictor and corrector also form the total acceleration from its parts)
void sg_seg_launch_predict(const sg_seg& s, double dt, hipStream_t st);
void sg_seg_launch_correct(const sg_seg& s, double dt, hipStream_t st);
void sg_seg_launch_morton_order(const sg_seg& s, hipStream_t st);
void sg_seg_launch_grav_sorted(const sg_seg& s, hipStream_t st);
void sg_seg_launch_grav_finish(const sg_seg& s, int with_pot, double G, double eps,
                               hipStream_t st);
// The neighbour build of every system, in the order of the per-system
// launches: the gas sort (grid rule, keys and counts, cell offsets, stable
// reorder and gather), the search, the scan of the neighbour counts into
// CSR offsets, the capacity check and the copy into the CSR rows.
void sg_seg_launch_sort(const sg_seg& s, hipStream_t st);
void sg_seg_launch_nbr_search(const sg_seg& s, hipStream_t st);
void sg_seg_launch_scan_nbr(const sg_seg& s, hipStream_t st);
void sg_seg_launch_nbr_finish(const sg_seg& s, hipStream_t st);
// Density, and the EOS records + FP32C forces on the predicted state
// (predicted != 0: vt, et) or the current one.
int64_t sg_sph_blocks(int64_t ng);
int sg_nbr_targets(int64_t ng);                // targets per wavefront of the search
int64_t sg_nbr_blocks(int64_t ng, int nt);
int64_t sg_compact_blocks(int64_t ng);
void sg_seg_launch_density(const sg_seg& s, hipStream_t st);
void sg_seg_launch_sph_state(const sg_seg& s, int predicted, hipStream_t st);

// Update and diagnostics.  Parts of the total acceleration (null: that part
// does not exist); predictor and corrector given them also write their sum
// to ax, ay, az, as sg_launch_combine does.
struct sg_acc_parts {
    const double *asx, *asy, *asz, *gx, *gy, *gz;
};
void sg_launch_predict(int64_t n, int64_t ng, double dt, double* x, double* y, double* z,
                       const double* vx, const double* vy, const double* vz, const double* e,
                       double* ax, double* ay, double* az, const double* dedt, double* vtx,
                       double* vty, double* vtz, double* et, const sg_acc_parts* parts,
                       hipStream_t st);
void sg_launch_correct(int64_t n, int64_t ng, double dt, double* vx, double* vy, double* vz,
                       double* e, const double* vtx, const double* vty, const double* vtz,
                       const double* et, double* ax, double* ay, double* az, const double* dedt,
                       const sg_acc_parts* parts, hipStream_t st);
void sg_launch_combine(int64_t n, int64_t ng, const sg_acc_parts& parts, double* ax, double* ay,
                       double* az, hipStream_t st);
size_t sg_diag_tmp_bytes();
void sg_launch_diagnostics(int64_t n, int64_t ng, const double* x, const double* y,
                           const double* z, const double* vx, const double* vy,
                           const double* vz, const double* m, const double* e,
                           const double* pot, double* tmp, double* out10, hipStream_t st);
