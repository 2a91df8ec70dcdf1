// pic_internal.h — device-side layout shared by the HIP kernels and the host driver of
// the particle hot path (gfx950).  Not part of the public C ABI (include/pic.h).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace pic {

constexpr int kGuard = 2;      // guard cells on each side of every grid axis (z: 0 in 2D)
constexpr int kMaxSpecies = 2;
constexpr int kBlock = 256;    // threads per workgroup of the particle kernels (4 wave64)
constexpr int kMjBins = 4096;  // reinjection sampler: bulk inverse-CDF bins
constexpr int kMjTail = 64;    // reinjection sampler: tail bins in -log2(1-p)

enum Frame { kPlain = 0, kShear = 1, kExpand = 2, kLeaky = 3, kShearExpand = 4 };
// frames with the shearing-box geometry, and with the expanding-box scale factors
constexpr bool frame_sheared(int f) { return f == kShear || f == kShearExpand; }
constexpr bool frame_expanding(int f) { return f == kExpand || f == kShearExpand; }

// Particle cells are packed as i | j << b0 | k << (b0+b1) with b_d = ceil(log2 n_d),
// so decoding is shifts and masks.  A dead particle has cell -1.
struct CellCode {
    int b0, b1;
    unsigned m0, m1;
    __host__ __device__ inline void decode(int32_t c, int& i, int& j, int& k) const
    {
        unsigned u = (unsigned)c;
        i = (int)(u & m0);
        j = (int)((u >> b0) & m1);
        k = (int)(u >> (b0 + b1));
    }
    __host__ __device__ inline int32_t encode(int i, int j, int k) const
    {
        return (int32_t)((unsigned)i | ((unsigned)j << b0) | ((unsigned)k << (b0 + b1)));
    }
};

// Geometry of the tile decomposition (power-of-two tile edges).
struct Tiles {
    int lt[3];    // log2 of the tile edge per axis
    int nt[3];    // tiles per axis
    int n_tiles;
    __host__ __device__ inline int key(int i, int j, int k) const
    {
        return (i >> lt[0]) + nt[0] * ((j >> lt[1]) + nt[1] * (k >> lt[2]));
    }
};

// Directions of the migration sort: (dx, dy, dz) in {-1,0,1}^3 between the tile a particle
// was sorted into and the tile of its new cell, index (dx+1) + 3 (dy+1) + 9 (dz+1); the last
// direction is the dead bin.  On an axis of two tiles the other tile is +1, whichever way.
// Beyond the x faces of the shearing box the y step is taken from the tile mig_center.
constexpr int kMigDirs = 28;
constexpr uint32_t kErrSort = 16u;  // a batched sort met a particle beyond the neighbour tiles
constexpr uint32_t kErrNoConverge = 32u;  // shearing-box sweeps missed their tolerance
constexpr int kMigStay = 13, kMigDead = 27;
// Tiles up to which the scatter's workgroups scan the tile totals themselves.  The sort of two species on 8 x 8
// tiles, us, so / with a scan launch: 289 tiles 14.9 / 17.0, 576 16.4 / 18.3, 1024 20.8 / 21.1.
constexpr int kMigSmall = 1024;
struct MigGeo {
    int nt[3], lt[3];
    int n_tiles;
    int many[3];  // -1 on an axis of several tiles, 0 on one of a single tile
    int general;  // an axis of two tiles, or of a size that is no multiple of the tile
    // shearing box: cells along y and, modulo them, the first row that the particles of tile 0 may
    // reach through the outer (first[1]) and the inner (first[0]) x face
    int shear, ny, first[2];
};

// The middle one of the (at most three) y tiles that the particles of y tile ty reach through an x
// face: they are T + 3 rows from ty T + first on (the row, one down or up by the move, one up or
// down by the fraction of Delta y_s).  On a ring of ny rows whose last tile has two rows or more,
// T + 3 rows touch three consecutive tiles at most.
__device__ inline int mig_center(const MigGeo& g, int ty, bool out)
{
    if (!g.shear || g.nt[1] <= 2) return ty;
    int r = (ty << g.lt[1]) + g.first[out ? 1 : 0];
    if (r >= g.ny) r -= g.ny;
    r = (r >> g.lt[1]) + 1;
    return r == g.nt[1] ? 0 : r;
}

// d in (-n, n) reduced on a ring of n tiles to -1, 0, +1, or 2 if it is farther
__device__ inline int ring_step(int d, int n)
{
    if (n <= 2) return n == 1 ? 0 : d & 1;
    const int r = d < 0 ? d + n : d;
    return r <= 1 ? r : (r == n - 1 ? -1 : 2);
}

__device__ inline void tile_coords(const MigGeo& g, int t, int& x, int& y, int& z)
{
    x = t % g.nt[0];
    const int r = t / g.nt[0];
    y = r % g.nt[1];
    z = r / g.nt[1];
}

// direction of a particle of source tile (sx, sy, sz) with new cell (x, y, z), or -1 if its new tile
// is not a neighbour; co, ci: the centres of sy beyond the outer and the inner x face
__device__ inline int mig_dir(const MigGeo& g, int sx, int sy, int sz, int co, int ci, int x, int y, int z)
{
    const int dx = ring_step((x >> g.lt[0]) - sx, g.nt[0]);
    const int tx = sx + dx;  // beyond a face: through it (a sheared box has three tiles in x or more)
    const int c = tx >= g.nt[0] ? co : (tx < 0 ? ci : sy);
    const int dy = ring_step((y >> g.lt[1]) - c, g.nt[1]);
    const int dz = ring_step((z >> g.lt[2]) - sz, g.nt[2]);
    if (dx == 2 || dy == 2 || dz == 2) return -1;
    return (dx + 1) + 3 * (dy + 1) + 9 * (dz + 1);
}
__device__ inline int mig_dir(const MigGeo& g, const CellCode& cc, int sx, int sy, int sz, int co, int ci, int32_t c)
{
    if (c < 0) return kMigDead;
    int x, y, z;
    cc.decode(c, x, y, z);
    return mig_dir(g, sx, sy, sz, co, ci, x, y, z);
}

// One species as seen by a push launch: input arrays (read through perm), output arrays
// (written in sorted slot order) and the unfused-deposit workspace.
struct SpeciesDev {
    const int32_t* cell_in;
    const float* off_in[3];
    const float* u_in[3];
    const uint32_t* id_in;
    const float* dr_in[3];
    int32_t* cell_out;
    float* off_out[3];
    float* u_out[3];
    uint32_t* id_out;
    float* dr_out[3];
    const int32_t* perm;  // sorted slot -> input index
    const int32_t* toff;  // tile offsets, n_tiles + 1
    int32_t* ws_cell;     // unfused deposit: old cell, old offsets, deposit displacement
    float* ws_off[3];
    float* ws_disp[3];
    float qm_hdt;         // (q/m) dt/2
    float q_dt;           // macro charge / dt
};

// Everything one push or deposit launch of one box needs, passed by value.
struct StepDev {
    int dim, frame;
    int n[3];
    CellCode cc;
    Tiles tl;
    int sy, sz;           // element strides of the guarded grid arrays (x stride 1)
    float* E[3];          // pointers to interior (0,0,0) of the guarded arrays
    float* B[3];
    float* J[3];
    float dt;
    // shearing box
    float sO;             // s Omega0
    float om_dt;          // Omega0 dt
    float alpha1;         // s Omega0 dt/2
    float half_nx;        // n[0]/2
    int dys_int;          // Delta y_s(t^{n+1}) = dys_int + dys_frac, dys_frac in [0,1)
    float dys_frac;
    // expanding box (Lambda at t^n, L^-1 at t^{n+1/2})
    float lam1p[3];       // 1 + Lambda_ii
    float ltil[3];        // (1 + Lambda_ii)/(1 - Lambda_ii)
    float tfac[3];        // 1/(1 - Lambda_ii)
    float linv[3];        // 1/l_i(t^{n+1/2})
    // leaky box
    int leaky_mode, use_3vec;
    int escape;  // the leaky box's escape rule applies (always in the leaky frame; on request
                 // in the shearing and expanding frames)
    float l_esc;
    uint32_t esc_thr;     // floor((dt/t_esc) 2^32)
    double g2thr;         // gamma_thr^2 - 1
    uint32_t key0, key1, step_lo, box_id;
    const float* mj;      // kMjBins + kMjTail values
    // fixed-point tile current: contribution * jscale -> integer units, units * junit -> J
    float jscale, junit;
    // a tile is shared out to 2^lsplit workgroups: by_species, the lowest bit names one of two species,
    // and part p of the others takes every 2^(lsplit - by_species)-th round of a species' slots
    int lsplit, by_species;
    // split tiles: the integer sums of each tile's parts and the count of those done (split_words), zero between
    // launches
    unsigned long long* tsum;
    // migration counts of the next sort, taken by the push: per species and source tile
    // (= this launch's tile), the particles per direction (mcnt[tile * kMigDirs + d], added to the
    // cleared counts by the parts of a split tile); a
    // particle beyond the neighbouring tiles sets mfb (the next sort is a radix sort then)
    int count_mig;
    int mig_latch;  // batched steps: latch kErrSort too
    MigGeo mg;
    uint32_t* mcnt[kMaxSpecies];
    int32_t* mfb[kMaxSpecies];
    // bookkeeping
    uint32_t* err;
    unsigned long long* ctr;  // [0] slow-path particles, [1] escapes
    int nsp;
    int track_ids;
    int count_sl;  // shearing box: count superluminal effective velocities (PIC_BOX_COUNT_SUPERLUMINAL)
    SpeciesDev sp[kMaxSpecies];
};

// Philox4x32-10 (Salmon, Moraes, Dror and Shaw, SC'11): ten rounds of the two 32x32->64
// multiplications with the published multipliers, key bumped by the published Weyl
// constants between rounds.
__device__ inline void philox4x32_10(uint32_t c[4], uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; r++) {
        const uint32_t a0 = c[0], a2 = c[2];
        const uint32_t hi0 = __umulhi(0xD2511F53u, a0), lo0 = 0xD2511F53u * a0;
        const uint32_t hi1 = __umulhi(0xCD9E8D57u, a2), lo1 = 0xCD9E8D57u * a2;
        c[0] = hi1 ^ c[1] ^ k0;
        c[1] = lo1;
        c[2] = hi0 ^ c[3] ^ k1;
        c[3] = lo0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
}

// Maps block b of a grid of nblk blocks to a work index so that each of the 8 XCDs (which
// receive blocks round-robin) processes one contiguous range of tiles and shares its L2
// for the overlapping tile halos.
__device__ inline int xcd_contiguous(int b, int nblk)
{
    const int x = b & 7, local = b >> 3;
    const int full = nblk >> 3, rem = nblk & 7;
    return x * full + (x < rem ? x : rem) + local;
}

// ---- batched launches
// One launch runs the blocks of many independent work units (boxes, or parts of boxes):
// prefix[u] is the first block of unit u, prefix[nu] the total.  A kernel body takes its unit's
// arguments, its block index inside the unit, the unit's block count and blockIdx.y.
struct UnitMap {
    const uint32_t* prefix;
    int nu;
};
__device__ inline int unit_of(const UnitMap& m, int b)  // the unit owning block b
{
    int lo = 0, hi = m.nu;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if ((int)m.prefix[mid] <= b)
            lo = mid;
        else
            hi = mid;
    }
    return __builtin_amdgcn_readfirstlane(lo);  // uniform: descriptor loads stay scalar
}
// name##_kernel(Args): one unit, arguments by value; name##_batch(table, map): many units (PIC_BATCH_KERNEL: these alone).
#define PIC_BATCH_KERNEL(name, Args, NT)                                                         \
    __global__ __launch_bounds__(NT) void name##_batch(const Args* __restrict__ t, UnitMap m)   \
    {                                                                                            \
        const int u = unit_of(m, (int)blockIdx.x);                                               \
        name##_body(t[u], (int)blockIdx.x - (int)m.prefix[u], (int)(m.prefix[u + 1] - m.prefix[u]), \
                    (int)blockIdx.y);                                                            \
    }
#define PIC_BATCHED_KERNEL(name, Args, NT)                                                       \
    __global__ __launch_bounds__(NT) void name##_kernel(Args a)                                  \
    {                                                                                            \
        name##_body(a, (int)blockIdx.x, (int)gridDim.x, (int)blockIdx.y);                        \
    }                                                                                            \
    PIC_BATCH_KERNEL(name, Args, NT)

// Geometry of a guarded grid array.
// Division of 32-bit unsigned integers by an invariant divisor d >= 1 (Granlund and Montgomery,
// "Division by invariant integers using multiplication", PLDI 1994, Fig. 4.1): with
// l = ceil(log2 d) and m = floor(2^32 (2^l - d) / d) + 1, q = (t1 + ((t - t1) >> 1)) >> (l - 1),
// t1 = mulhi(m, t), for every t < 2^32 and d >= 2; d = 1 is q = t.
struct FastDiv {
    uint32_t m;
    int l;  // 0 for d = 1
    static FastDiv make(uint32_t d)
    {
        FastDiv f{0u, 0};
        while ((1ull << f.l) < d) f.l++;
        if (f.l > 0)
            f.m = (uint32_t)((((1ull << 32) * ((1ull << f.l) - d)) / d) + 1ull);
        return f;
    }
    __device__ inline uint32_t div(uint32_t t) const
    {
        if (l == 0) return t;
        const uint32_t t1 = __umulhi(m, t);
        return (t1 + ((t - t1) >> 1)) >> (l - 1);
    }
};

struct GridDev {
    int dim;
    int n[3];
    int g[3];    // guard width per axis
    int sy, sz;  // element strides (x stride 1)
    FastDiv div0, div1;  // division by n[0] and by n[1] (linear interior index -> x, y, z)
    FastDiv divyg;       // division by the guarded row count n[1] + 2 g[1]
};

// One Yee update: X_i <- fout_i (fin_i X_i +/- dt curl(g Y)_i [- 4 pi dt J_i]).
struct MaxwellDev {
    GridDev G;
    float* E[3];
    float* B[3];
    const float* J[3];
    float dt;
    float fin[3], fout[3], gf[3];
};

// Arguments of the grid kernels (one unit each; batched launches take tables of them).
struct Comp6 {
    float* p[6];
};
struct Comp3 {
    float* p[3];
};
struct FillArgs {  // guard fill of ncomp = gridDim.y arrays
    GridDev G;
    Comp6 A;
    int shear, dys_int;
    float dys_w;
    uint32_t n[3];  // guard cells of the x, y and z slabs
};
struct FoldPArgs {  // periodic current fold, in place
    GridDev G;
    Comp3 J;
    uint32_t n[3];  // cells of the x layers, of the y layers and of the z layers, each without the former
    int x0;         // columns x0 .. x0 + wx - 1 of the y and z layers
    uint32_t wx;
};
struct ShearFoldArgs {  // J' transport along y and shearing-periodic x fold, in -> out
    GridDev G;
    Comp3 in, out;
    float sO_hdt, half_nx;
    int dys_int;
    float dys_w;
};
// What a push starts from: the current arrays (n words each), the fallback flags and, for split
// tiles, the migration counts (nm words) at zero.
struct ClearArgs {
    float* J[3];
    int64_t n;
    int32_t* flag[kMaxSpecies];
    uint32_t* mcnt[kMaxSpecies];
    int64_t nm;
};
struct ZeroArgs {  // n 32-bit words set to zero
    uint32_t* p;
    int64_t n;
};

// One fixed-point sweep of the shearing-box implicit midpoint rule: Fo = C + dt/2 L(Fk); the
// first sweep of a step (Fk = F^n) also writes C = F^n + dt/2 L(F^n) - 4 pi dt J'.
struct KsbDev {
    GridDev G;
    const float* Fk[6];  // iterate, Bx By Bz Ex Ey Ez (the interior is read)
    float* C[6];         // constant part of the step (written by the first sweep)
    float* Fo[6];        // next iterate (interior)
    const float* J[3];
    float dt, sO, half_nx;
    // shift of the iterate's shearing-periodic x images, Delta y_s = ydys_int + ydys_w with
    // ydys_w in [0,1): the sweeps read the cells beyond the x faces there, not from guard cells
    int ydys_int;
    float ydys_w;
    // tolerance mode (conv != nullptr): sweep k adds max|F^{k+1} - F^k| and max|F^{k+1}| (FP32
    // bit patterns, non-negative, so unsigned order is float order; NaN counts as +inf) into the
    // pairs at conv + kConvSweep k, which start at zero; it returns at once when the sweep before it
    // met the tolerance, leaving its pairs at zero, which reads as met for the next one
    uint32_t* conv;
    float tol;
    int k;
    // two sweeps per pass or launch (fixed sweep count): the shift of the
    // intermediate iterate's x images, Delta y_s at t^{n+1} = y1_int + y1_w
    int y1_int;
    float y1_w;
    int zc;  // planes per workgroup of the staged kernels (set by their launchers)
    // combined shearing and expanding frame (sweeps of one thread per cell, one or two a launch): the iterates are
    // the expanding-frame fields, the curls act on dfac[c] F_c and kz multiplies the z
    // transport of E'_y in dE'_z/dt
    int expand;
    float dfac[3];
    float kz;
};
constexpr int kKsbMaxSweeps = 64;
// A sweep's pair of maxima is kept in kConvSlots places of a cache line each, workgroup b adding to
// place b % kConvSlots: at one place the atomics of 2048 workgroups took 24 us of a sweep that
// itself takes 11 (128 x 64 x 64 cells).
constexpr int kConvSlots = 16, kConvStride = 32, kConvSweep = kConvSlots * kConvStride;
// words of a box's convergence record: kKsbMaxSweeps sweeps, then the sweep count of the last
// step
constexpr int kKsbConvWords = kConvSweep * kKsbMaxSweeps + 2;

// End of a tolerance-mode step: k* = the first sweep that met the tolerance (the last sweep K-1
// if none did, which latches kErrNoConverge).  The iterate of sweep k* sits in the field set
// that sweep K-1 would have written when K-1-k* is even, in the other set otherwise: then
// the interior of src (that other set) is copied to dst.
struct KsbFin {
    GridDev G;
    const uint32_t* conv;
    int32_t* sweeps;
    uint32_t* err;
    float tol;
    int K;
    const float* src[6];
    float* dst[6];
};

// Sort workspace of one species.
struct SortBufs {
    uint32_t* keys[2];
    uint32_t* vals[2];
    uint32_t* hist;
    uint32_t* scratch;
    // migration sort (kMigDirs counters per source tile, per-destination scans)
    uint32_t* mcnt;    // n_tiles * kMigDirs: particles of source tile s moving in direction d
    uint32_t* mpre;    // n_tiles * kMigDirs: offset of (s, d) inside its destination tile
    uint32_t* tot;     // n_tiles + 1: particles arriving in each tile (last entry 0)
    uint32_t* start;   // n_tiles + 1: exclusive scan of tot
    uint32_t* dcnt;    // n_tiles + 1: particles of each source tile that died (last entry 0)
    uint32_t* dpre;    // n_tiles + 1: exclusive scan of dcnt
    uint32_t* mscratch;
    int32_t* fallback; // set when a particle left the neighbourhood the migration sort covers
};

// Migration sort of one species: its arrays, the push's counts, and the general sort's buffers for
// a species that turns out to be beyond it
struct MigArgs {
    const int32_t* cell;
    const int32_t* toff_prev;
    int n_upper, which;  // which: the vals buffer that takes the permutation
    CellCode cc;
    MigGeo g;
    const uint32_t* mcnt;
    uint32_t *mpre, *tot, *dcnt, *start, *dpre;
    uint32_t *keys[2], *vals[2];
    int32_t *toff, *n_live;
    const int32_t* fallback;
    unsigned long long* n_fallback;
};
struct MigPair {
    MigArgs s[kMaxSpecies];
};

// ---- launchers (gpd.hip, sort.hip, grid.hip, xfer.hip)
bool tile_shape_supported(int dim, const int t[3]);
// share the tiles of a push or deposit out to workgroups (lsplit, by_species): n_tiles tiles in the launch
// (of all its boxes), whole_tiles tiles' worth of cells, slots_per_tile slots of the fuller species a tile on average in this one
void split_tiles(StepDev& P, const int t[3], int64_t n_tiles, int64_t whole_tiles, int64_t slots_per_tile);
// 64-bit words that the parts' sums need for a box of n_tiles tiles
int64_t split_words(int dim, const int t[3], int64_t n_tiles);
// supported tile shapes (batched: those of the batched launch); the default shape comes first
int tile_candidates(int dim, bool batched, int (*out)[3], int max);
hipError_t launch_gather_push(const StepDev& P, const int t[3], int fuse, hipStream_t st);
hipError_t launch_deposit(const StepDev& P, const int t[3], hipStream_t st);
// fused push of many boxes of one dimension, tile shape and frame (table: one StepDev per box,
// m.prefix: first block of each box = its first tile)
bool batch_tile_supported(int dim, const int t[3]);
hipError_t launch_gather_push_batch(const StepDev* table, UnitMap m, int blocks, int dim,
                                    const int t[3], int frame, hipStream_t st);

size_t scan_scratch_words(int64_t n);
size_t sort_hist_words(int64_t n);
hipError_t tile_sort(const int32_t* cell, const int32_t* n_live_in, int n_upper, CellCode cc,
                     Tiles tl, SortBufs& sb, int32_t* toff, int32_t* n_live_out, int& which,
                     hipStream_t st);

// Migration sort: stable counting sort by tile of arrays still grouped by the tiles of the
// previous sort (toff_prev), every particle within one tile of its old one, the counts taken by the
// push.  Writes the permutation to vals[which] and the offsets to toff.
size_t migrate_scratch_words(int n_tiles);
hipError_t migrate_sort(const MigPair& a, int n_species, uint32_t* const* scratch, hipStream_t st);
unsigned mig_offset_blocks(int n_tiles);
bool mig_needs_scan(int n_tiles);

// batched launches of the grid and sort kernels (tables of per-unit arguments on the device)
// per-component factors of a field set (the combined frame's conversion to and from the
// expanding-frame fields): F_c *= f[c % 3] on the interior
struct ScaleArgs {
    GridDev G;
    float* F[6];
    float f[3];
};
enum GridBatchKind {
    kBatchZero, kBatchFill, kBatchFoldP, kBatchShearFold, kBatchYeeB, kBatchYeeE,
    kBatchKsbFirst, kBatchKsbNext, kBatchKsbPairFirst, kBatchKsbPairNext, kBatchKsbFinal, kBatchScale
};
hipError_t grid_batch(GridBatchKind k, const void* table, UnitMap m, int blocks, int ydim,
                      hipStream_t st);
unsigned grid_blocks(int64_t items);  // workgroups of kBlock threads for one item per thread
enum SortBatchKind { kBatchMigOffsets, kBatchMigScan, kBatchMigScatter };
hipError_t sort_batch(SortBatchKind k, const void* table, UnitMap m, int blocks, hipStream_t st);
int sort_result_buffer(const Tiles& tl);  // sort buffer holding the sorted pairs

FillArgs fill_args(const GridDev& G, float* const* comps, int ncomp, int shear, double dys);
unsigned fill_blocks(const FillArgs& a);
hipError_t fill_guards(const GridDev& G, float* const* comps, int ncomp, int shear, double dys,
                       hipStream_t st);
// Fold the current guards (y, z periodic).  Shearing box: with the J' transport and the
// shearing-periodic x fold in one pass from J into `out` (the caller then swaps the two arrays);
// otherwise periodic in place.
FoldPArgs fold_args(const GridDev& G, float* const* J, int shear);
unsigned fold_blocks(const FoldPArgs& a);
unsigned shear_fold_blocks(const GridDev& G);
hipError_t fold_current(const GridDev& G, float* const* J, float* const* out, int shear,
                        double sO, double dt, double dys_half, hipStream_t st);
hipError_t yee_b(const MaxwellDev& M, hipStream_t st);
hipError_t yee_e(const MaxwellDev& M, hipStream_t st);
// one sweep, one thread per cell: any grid, any sheared frame; the cells beyond the faces are read at their images
// (as by the kernels below)
hipError_t ksb_sweep(const KsbDev& K, bool first, hipStream_t st);
// the staged sweep: large 3D grids whose x size is a multiple of its column tile (128), the shearing box
bool ksb_staged(const GridDev& G);
hipError_t ksb_sweep_staged(const KsbDev& K, bool first, hipStream_t st);
// two sweeps per launch (fixed sweep count, K.y1_*): small grids of any shape, any sheared frame
bool ksb_pairs(const GridDev& G);
unsigned ksb_pair_blocks(const GridDev& G);
hipError_t ksb_pair(const KsbDev& K, bool first, hipStream_t st);
// the two-sweep pass applies: a large grid whose arrays span less than 4 GiB (32-bit offsets)
bool ksb_pass_fits(const GridDev& G);
// two sweeps F^k -> F^{k+2} in one pass over memory (large 3D grids); first: F^k = F^n,
// the pass also writes C
hipError_t ksb_pass(const KsbDev& K, bool first, hipStream_t st);

hipError_t ksb_finalize(const KsbFin& F, hipStream_t st);
// interior of six field components (B then E) times f[c % 3]
hipError_t scale_fields(const GridDev& G, float* const* F, const float f[3], hipStream_t st);
constexpr int kKsbFinBlocks = 512;  // workgroups per box of the finalize copy (grid stride)
hipError_t zero_floats(float* p, int64_t n, hipStream_t st);
hipError_t clear_for_push(const ClearArgs& a, hipStream_t st);
hipError_t interior_copy(const GridDev& G, float* const* guarded, float* const* dense, int ncomp, int to_dense,
                         hipStream_t st);
constexpr int kPartSums = 7;       // rows per species: gamma-1, u (3), u_c^2/gamma (3)
// the particles and counters that a box's record is taken from, and the record
struct SumArgs {
    struct Species {
        const int32_t* cell;  // null: a box without escapes
        const float* u[3];
        const int32_t* n_live;
    } s[kMaxSpecies];
    int nsp;
    const unsigned long long* ctr;
    const uint32_t* err;
    const int32_t* sweeps;  // null: known to the host
};
struct BoxRecord {
    double row[6 + kPartSums * kMaxSpecies];  // squares of B, E; then per species kPartSums sums
    unsigned long long ctr[4];
    int32_t live[kMaxSpecies];
    uint32_t err;
    int32_t sweeps;
};
// part: one row of nblk partials for every row of the record
hipError_t box_record(const GridDev& G, float* const* comps, const SumArgs& P, double* part, int nblk, BoxRecord* out,
                      hipStream_t st);
constexpr int kHistMaxBins = 4096;  // energy_histogram
hipError_t energy_histogram(const int32_t* cell, const float* ux, const float* uy, const float* uz,
                            const int32_t* n_live, const double* edges, int nbins,
                            unsigned long long* counts, hipStream_t st);

// Static device scratch of the entry points that allocate nothing (noalloc.hip): the current
// device's copy of one file-scope array of kStaticScratchBytes, its address taken once per
// device.  The histogram variant keeps its edges (FP64, kHistMaxBins + 1) at the start and its
// counts (uint64, kHistMaxBins + 2) at kStaticHistCountsOffset.
constexpr size_t kStaticHistCountsOffset = ((size_t)(kHistMaxBins + 1) * 8 + 255) & ~(size_t)255;
constexpr size_t kStaticScratchBytes =
    (kStaticHistCountsOffset + (size_t)(kHistMaxBins + 2) * 8 + 255) & ~(size_t)255;
hipError_t static_scratch(void** ptr, size_t* bytes);

// particles between the boundary layout (dense arrays: off[c * n + i], u, dr likewise; linear cells)
// and a species' arrays; null pointers are left out
struct Particles {
    int32_t* cell;
    float* off[3];
    float* u[3];
    uint32_t* id;
    float* dr[3];
};
hipError_t particles_in(const Particles& to, int64_t n, const int32_t* cell, const float* off, const float* u,
                        const uint32_t* id, const float* dr, int dim, const GridDev& G, CellCode cc, int32_t* n_live,
                        uint32_t* err, hipStream_t st);
// the *n_live particles (at most n_upper) out; dr: ndr components, the others 0
hipError_t particles_out(const Particles& from, const int32_t* n_live, int64_t n_upper, int32_t* cell, float* off,
                         float* u, uint32_t* id, float* dr, int dim, int ndr, const GridDev& G, CellCode cc,
                         hipStream_t st);
hipError_t device_copy16(void* dst, const void* src, int64_t nwords, hipStream_t st);

}  // namespace pic
