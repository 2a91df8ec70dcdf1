// sort.hip — stable tile counting sort of the particle arrays (gfx950).
//
// key = tile of the particle's cell (dead particles and slots beyond the live count go to a
// dead bin = n_tiles).  The sort is a stable LSD radix sort of (key, index) pairs with 8-bit
// digits: per-chunk digit histograms, one exclusive scan in digit-major order, and a stable
// scatter that ranks equal digits inside a wave with 8 ballots and a popcount.  The sorted
// indices are the permutation the push kernel reads its particles through, so the particle
// payload itself is moved only once, by the push.  Tile offsets come from the sorted keys.
#include "pic_internal.h"

namespace pic {

constexpr int kItems = 16;                // items per thread per chunk
constexpr int kChunk = kBlock * kItems;   // 4096 items per block


__global__ __launch_bounds__(kBlock) void make_keys_kernel(const int32_t* __restrict__ cell,
                                                           const int32_t* __restrict__ n_live,
                                                           int n_upper, CellCode cc, Tiles tl,
                                                           uint32_t* __restrict__ keys,
                                                           uint32_t* __restrict__ vals)
{
    const int nl = *n_live;
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < n_upper; i += gridDim.x * kBlock) {
        uint32_t k = (uint32_t)tl.n_tiles;
        if (i < nl) {
            const int32_t c = cell[i];
            if (c >= 0) {
                int x, y, z;
                cc.decode(c, x, y, z);
                k = (uint32_t)tl.key(x, y, z);
            }
        }
        keys[i] = k;
        vals[i] = (uint32_t)i;
    }
}

// chunks of kChunk keys, a grid-stride loop over them
__global__ __launch_bounds__(kBlock) void radix_hist_kernel(const uint32_t* __restrict__ keys,
                                                            int n, int nchunks, int shift,
                                                            uint32_t* __restrict__ hist)
{
    __shared__ uint32_t cnt[256];
    const int tid = threadIdx.x;
    for (int ch = blockIdx.x; ch < nchunks; ch += gridDim.x) {
        cnt[tid] = 0;
        __syncthreads();
        const int base = ch * kChunk;
#pragma unroll 4
        for (int r = 0; r < kItems; r++) {
            const int i = base + r * kBlock + tid;
            if (i < n) atomicAdd(&cnt[(keys[i] >> shift) & 255u], 1u);
        }
        __syncthreads();
        hist[tid * nchunks + ch] = cnt[tid];
        __syncthreads();
    }
}

__global__ __launch_bounds__(kBlock) void radix_scatter_kernel(
    const uint32_t* __restrict__ kin, const uint32_t* __restrict__ vin, int n, int nchunks,
    int shift, const uint32_t* __restrict__ hscan, uint32_t* __restrict__ kout,
    uint32_t* __restrict__ vout)
{
    __shared__ uint32_t base[256];
    __shared__ uint32_t wcnt[4][256];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const unsigned long long lt = (1ull << lane) - 1ull;
    for (int b = blockIdx.x; b < nchunks; b += gridDim.x) {
        base[tid] = hscan[tid * nchunks + b];
        for (int r = 0; r < kItems; r++) {
            wcnt[0][tid] = wcnt[1][tid] = wcnt[2][tid] = wcnt[3][tid] = 0;
            __syncthreads();
            const int i = b * kChunk + r * kBlock + tid;
            const bool valid = i < n;
            const uint32_t key = valid ? kin[i] : 0u;
            const uint32_t val = valid ? vin[i] : 0u;
            const uint32_t d = (key >> shift) & 255u;
            unsigned long long m = __ballot(valid);
#pragma unroll
            for (int bit = 0; bit < 8; bit++) {
                const bool on = (d >> bit) & 1u;
                const unsigned long long bb = __ballot(on);
                m &= on ? bb : ~bb;
            }
            const int rank = __popcll(m & lt);
            if (valid && rank == 0) wcnt[w][d] = (uint32_t)__popcll(m);
            __syncthreads();
            if (valid) {
                uint32_t pre = 0;
                for (int k = 0; k < w; k++) pre += wcnt[k][d];
                const uint32_t pos = base[d] + pre + (uint32_t)rank;
                kout[pos] = key;
                vout[pos] = val;
            }
            __syncthreads();
            base[tid] += wcnt[0][tid] + wcnt[1][tid] + wcnt[2][tid] + wcnt[3][tid];
            __syncthreads();
        }
    }
}

// off[t] = first sorted position with key >= t, t in [0, n_tiles+1]; off[n_tiles] is the live
// count (dead bin starts there), off[n_tiles+1] = n.
__global__ __launch_bounds__(kBlock) void offsets_kernel(const uint32_t* __restrict__ keys, int n,
                                                         int n_tiles, int32_t* __restrict__ off,
                                                         int32_t* __restrict__ n_live)
{
    const int stride = gridDim.x * kBlock;
    if (n == 0) {
        for (int i = blockIdx.x * kBlock + threadIdx.x; i <= n_tiles + 1; i += stride) off[i] = 0;
        if (blockIdx.x == 0 && threadIdx.x == 0) *n_live = 0;
        return;
    }
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += stride) {
        const int k = (int)keys[i];
        const int kp = i > 0 ? (int)keys[i - 1] : -1;
        for (int t = kp + 1; t <= k; t++) {
            off[t] = i;
            if (t == n_tiles) *n_live = i;
        }
        if (i == n - 1) {
            for (int t = k + 1; t <= n_tiles + 1; t++) {
                off[t] = n;
                if (t == n_tiles) *n_live = n;
            }
        }
    }
}

// ------------------------------------------------------------------ exclusive scan (uint32)
__device__ inline uint32_t wave_incl_scan(uint32_t v)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(v, o, 64);
        if (lane >= o) v += t;
    }
    return v;
}

__global__ __launch_bounds__(kBlock) void scan_blocks_kernel(const uint32_t* in, uint32_t* out,
                                                             int n, uint32_t* bsum)
{
    __shared__ uint32_t s[kChunk];
    __shared__ uint32_t ws[4];
    const int tid = threadIdx.x;
    const int64_t base = (int64_t)blockIdx.x * kChunk;
    for (int k = 0; k < kItems; k++) {
        const int e = k * kBlock + tid;
        s[e] = base + e < n ? in[base + e] : 0u;
    }
    __syncthreads();
    uint32_t loc[kItems];
    uint32_t sum = 0;
#pragma unroll
    for (int j = 0; j < kItems; j++) {
        loc[j] = s[tid * kItems + j];
        sum += loc[j];
    }
    const uint32_t inc = wave_incl_scan(sum);
    const int w = tid >> 6, lane = tid & 63;
    if (lane == 63) ws[w] = inc;
    __syncthreads();
    uint32_t run = inc - sum;
    for (int k = 0; k < w; k++) run += ws[k];
    const uint32_t tot = ws[0] + ws[1] + ws[2] + ws[3];
#pragma unroll
    for (int j = 0; j < kItems; j++) {
        s[tid * kItems + j] = run;
        run += loc[j];
    }
    __syncthreads();
    for (int k = 0; k < kItems; k++) {
        const int e = k * kBlock + tid;
        if (base + e < n) out[base + e] = s[e];
    }
    if (tid == 0 && bsum) bsum[blockIdx.x] = tot;
}

__global__ __launch_bounds__(kBlock) void scan_add_kernel(uint32_t* out, int n,
                                                          const uint32_t* bpre)
{
    const int64_t i = (int64_t)blockIdx.x * kChunk;
    const uint32_t add = bpre[blockIdx.x];
    for (int k = 0; k < kItems; k++) {
        const int64_t e = i + k * kBlock + threadIdx.x;
        if (e < n) out[e] += add;
    }
}

// words of scratch the scan of n items needs
size_t scan_scratch_words(int64_t n)
{
    size_t w = 0;
    while (n > 1) {
        n = (n + kChunk - 1) / kChunk;
        w += 2 * (size_t)n + 64;
    }
    return w + 64;
}

static hipError_t scan_exclusive(const uint32_t* in, uint32_t* out, int n, uint32_t* scratch,
                                 hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const int nblk = (n + kChunk - 1) / kChunk;
    uint32_t* bsum = scratch;
    uint32_t* bpre = scratch + nblk;
    scan_blocks_kernel<<<nblk, kBlock, 0, st>>>(in, out, n, nblk > 1 ? bsum : nullptr);
    if (nblk > 1) {
        hipError_t e = scan_exclusive(bsum, bpre, nblk, scratch + 2 * nblk + 64, st);
        if (e != hipSuccess) return e;
        scan_add_kernel<<<nblk, kBlock, 0, st>>>(out, n, bpre);
    }
    return hipGetLastError();
}

size_t sort_hist_words(int64_t n) { return 256 * (size_t)((n + kChunk - 1) / kChunk) + 64; }

// grid of the radix kernels: enough workgroups to fill the chip, loops beyond
static unsigned grid_cap(int blocks) { return (unsigned)(blocks < 4096 ? (blocks > 0 ? blocks : 1) : 4096); }

static int radix_passes(const Tiles& tl)
{
    int bits = 0;
    while ((1u << bits) <= (unsigned)tl.n_tiles) bits++;
    return (bits + 7) / 8;
}

// Stable sort by tile; returns the buffer index (0/1) holding the sorted (key, index) pairs.
hipError_t tile_sort(const int32_t* cell, const int32_t* n_live_in, int n_upper, CellCode cc,
                     Tiles tl, SortBufs& sb, int32_t* toff, int32_t* n_live_out, int& which,
                     hipStream_t st)
{
    which = 0;
    if (n_upper > 0) {
        make_keys_kernel<<<grid_cap((n_upper + kBlock - 1) / kBlock), kBlock, 0, st>>>(
            cell, n_live_in, n_upper, cc, tl, sb.keys[0], sb.vals[0]);
        const int passes = radix_passes(tl);
        const int nchunks = (n_upper + kChunk - 1) / kChunk;
        for (int p = 0; p < passes; p++) {
            const int shift = 8 * p;
            radix_hist_kernel<<<grid_cap(nchunks), kBlock, 0, st>>>(sb.keys[which], n_upper,
                                                                     nchunks, shift, sb.hist);
            hipError_t e = scan_exclusive(sb.hist, sb.hist, 256 * nchunks, sb.scratch, st);
            if (e != hipSuccess) return e;
            radix_scatter_kernel<<<grid_cap(nchunks), kBlock, 0, st>>>(
                sb.keys[which], sb.vals[which], n_upper, nchunks, shift, sb.hist,
                sb.keys[which ^ 1], sb.vals[which ^ 1]);
            which ^= 1;
        }
    }
    const int nb = ((n_upper > tl.n_tiles + 2 ? n_upper : tl.n_tiles + 2) + kBlock - 1) / kBlock;
    offsets_kernel<<<grid_cap(nb), kBlock, 0, st>>>(sb.keys[which], n_upper, tl.n_tiles, toff,
                                                    n_live_out);
    return hipGetLastError();
}

// ------------------------------------------------------------------ migration sort
// Between two sorts a particle moves less than one cell, so the particles of source tile s
// (the slots toff_prev[s] .. toff_prev[s+1]-1, in the order of the previous sort) land in s or
// one of its neighbours.  The stable counting sort by the new tile then needs, per source tile,
// only the counts per direction (kMigDirs of them, taken by the push) instead of a radix sort:
//   offsets: per destination tile, its sources in increasing tile order give each
//            (source, direction) pair its offset inside the destination, and the total;
//   scan:    destination starts (= the new tile offsets) and the dead bin's per-source starts (by
//            the scatter's workgroups themselves on small tile grids);
//   scatter: per source tile, in slot order, stable ranks per direction.
// Both species take each of the two or three launches together.
// The result equals the stable radix sort: within a destination tile the particles come in
// increasing source tile, i.e. increasing slot, for the live slots (the permutation's
// observable part).  Slots from the previous dead bin stay dead at the end, after the
// particles that died since.  A push that meets a particle beyond the neighbouring tiles (none of
// its own moves does: only one that the caller moved in its memory between sort and push) sets a
// flag, on which the scatter's first workgroup sorts the species alone.

__device__ inline void dir_steps(int d, int& dx, int& dy, int& dz)
{
    dx = d % 3 - 1;
    dy = (d / 3) % 3 - 1;
    dz = d / 9 - 1;
}

__device__ inline bool step_possible(int n, int d) { return n > 2 || (n == 2 ? d >= 0 : d == 0); }
__device__ inline bool dir_possible(const MigGeo& g, int dx, int dy, int dz)
{
    return step_possible(g.nt[0], dx) && step_possible(g.nt[1], dy) && step_possible(g.nt[2], dz);
}

__device__ inline int wrap_tile(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }

// tile reached from source (sx, sy, sz) in direction (dx, dy, dz)
__device__ inline int mig_dst(const MigGeo& g, int sx, int sy, int sz, int dx, int dy, int dz)
{
    const int tx = sx + dx;
    const int c = tx >= g.nt[0] ? mig_center(g, sy, true) : (tx < 0 ? mig_center(g, sy, false) : sy);
    return wrap_tile(tx, g.nt[0]) +
           g.nt[0] * (wrap_tile(c + dy, g.nt[1]) + g.nt[1] * wrap_tile(sz + dz, g.nt[2]));
}

// source tile that reaches (tx, ty, tz) in direction (dx, dy, dz), -1 if there is none.  Beyond an
// x face of the shearing box y tiles are taken from the face's centre, which on a y size that is
// no multiple of the tile is sy + (the centre of tile 0) + e, e = 0 or 1: one candidate for each e.
__device__ inline int mig_src(const MigGeo& g, int tx, int ty, int tz, int dx, int dy, int dz, int e)
{
    const int sx = tx - dx, m = wrap_tile(ty - dy, g.nt[1]);
    int sy = m;
    if (g.shear && g.nt[1] > 2 && (sx < 0 || sx >= g.nt[0])) {
        const bool out = sx < 0;  // the source sits at the outer end and left through the outer face
        sy = wrap_tile(m - mig_center(g, 0, out) - e, g.nt[1]);
        if (sy < 0) sy += g.nt[1];
        if (mig_center(g, sy, out) != m) return -1;
    } else if (e) {
        return -1;
    }
    return wrap_tile(sx, g.nt[0]) + g.nt[0] * (sy + g.nt[1] * wrap_tile(tz - dz, g.nt[2]));
}

// One wave per destination tile; lanes 0 .. 26 take a direction each, lanes 27 .. 53 the second
// candidates.  Away from the faces the sources in increasing tile order are the directions in
// decreasing order: a wave scan gives the offsets (27 rounds of shuffles otherwise).
__device__ __attribute__((always_inline)) inline void mig_offsets_body(const MigArgs& a, int blk, int, int)
{
    if (*a.fallback) return;
    const MigGeo& g = a.g;
    const int lane = threadIdx.x & 63;
    const int t = blk * (kBlock / 64) + (threadIdx.x >> 6);
    if (t == 0 && lane == 0) {
        a.tot[g.n_tiles] = 0;
        a.dcnt[g.n_tiles] = 0;
    }
    if (t >= g.n_tiles) return;
    int tx, ty, tz;
    tile_coords(g, t, tx, ty, tz);
    const int e = lane >= 27 ? 1 : 0, dir = lane - 27 * e;
    uint32_t c = 0;
    int src = -1;
    if (lane < 54) {
        int dx, dy, dz;
        dir_steps(dir, dx, dy, dz);
        if (dir_possible(g, dx, dy, dz)) src = mig_src(g, tx, ty, tz, dx, dy, dz, e);
        if (src >= 0) c = a.mcnt[(size_t)src * kMigDirs + dir];
    }
    // the particles that stay: the tile's particles less all others
    uint32_t leave = lane < kMigDirs && lane != kMigStay ? a.mcnt[(size_t)t * kMigDirs + lane] : 0u;
    const uint32_t dead = __shfl(leave, kMigDead, 64);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) leave += __shfl_xor(leave, o, 64);
    if (lane == kMigStay) c = (uint32_t)(a.toff_prev[t + 1] - a.toff_prev[t]) - leave;
    uint32_t pre = 0, total;
    const bool inner = tx > 0 && tx < g.nt[0] - 1 && ty > 0 && ty < g.nt[1] - 1 &&
                       (g.nt[2] == 1 || (tz > 0 && tz < g.nt[2] - 1));
    if (inner) {  // sum over the lanes above
        uint32_t inc = c;
#pragma unroll
        for (int o = 1; o < 32; o <<= 1) {
            const uint32_t v = __shfl_down(inc, o, 64);
            if (lane + o < 27) inc += v;
        }
        pre = inc - c;
        total = __shfl(inc, 0, 64);
    } else {
        const int key = src >= 0 ? src : 0x7fffffff;
        total = 0;
        for (int k = 0; k < (g.shear ? 54 : 27); k++) {
            const int kk = __shfl(key, k, 64);
            const uint32_t ck = __shfl(c, k, 64);
            total += ck;
            if (kk < key) pre += ck;
        }
    }
    if (src >= 0) a.mpre[(size_t)src * kMigDirs + dir] = pre;
    if (lane == 0) {
        a.tot[t] = total;
        a.dcnt[t] = dead;
    }
}
PIC_BATCH_KERNEL(mig_offsets, MigArgs, kBlock)

// Exclusive scans of the arrivals and of the dead per tile, one workgroup each, 16 words a thread
// and round.
constexpr int kScanBlock = 1024, kScanItems = 16;
__device__ __attribute__((always_inline)) inline void mig_scan_body(const MigArgs& a, int blk, int, int)
{
    if (*a.fallback) return;
    const uint32_t* __restrict__ in = blk == 0 ? a.tot : a.dcnt;
    uint32_t* __restrict__ out = blk == 0 ? a.start : a.dpre;
    const int n = a.g.n_tiles + 1, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    __shared__ uint32_t ws[kScanBlock / 64];
    uint32_t carry = 0;
    for (int base = 0; base < n; base += kScanBlock * kScanItems) {
        const int i0 = base + tid * kScanItems;
        uint32_t v[kScanItems], sum = 0;
#pragma unroll
        for (int k = 0; k < kScanItems; k++) v[k] = i0 + k < n ? in[i0 + k] : 0u;
#pragma unroll
        for (int k = 0; k < kScanItems; k++) sum += v[k];
        const uint32_t inc = wave_incl_scan(sum);
        if (lane == 63) ws[w] = inc;
        __syncthreads();
        uint32_t run = carry + inc - sum, all = 0;
#pragma unroll
        for (int k = 0; k < kScanBlock / 64; k++) {
            if (k < w) run += ws[k];
            all += ws[k];
        }
        carry += all;
#pragma unroll
        for (int k = 0; k < kScanItems; k++) {
            if (i0 + k < n) out[i0 + k] = run;
            run += v[k];
        }
        __syncthreads();
    }
}
PIC_BATCH_KERNEL(mig_scan, MigArgs, kScanBlock)

// The whole sort by one workgroup (a particle was found beyond the neighbouring tiles): stable LSD
// radix passes over (key, slot), 8 bits each, as the general sort does with many workgroups.  Only a caller
// that moves particles in its memory between sort and push comes here; it saves every other step the gated
// launches of the general sort, and costs that one 12 ms a million particles (two digits).
__device__ __attribute__((always_inline)) inline void radix_alone(const MigArgs& a, uint32_t* lds)
{
    uint32_t* const base = lds;  // 256 words, then 256 a wave, then one a wave
    uint32_t(*const wcnt)[256] = reinterpret_cast<uint32_t(*)[256]>(lds + 256);
    uint32_t* const ws = lds + 256 * (1 + kBlock / 64);
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, n = a.n_upper, nt = a.g.n_tiles;
    const int nl = a.toff_prev[nt];
    const unsigned long long lt = (1ull << lane) - 1ull;
    for (int i = tid; i < n; i += kBlock) {
        const int32_t c = i < nl ? a.cell[i] : -1;
        int x, y, z;
        a.cc.decode(c, x, y, z);
        a.keys[0][i] = c < 0 ? (uint32_t)nt
                             : (uint32_t)((x >> a.g.lt[0]) + a.g.nt[0] * ((y >> a.g.lt[1]) + a.g.nt[1] * (z >> a.g.lt[2])));
        a.vals[0][i] = (uint32_t)i;
    }
    __syncthreads();
    int in = 0;
    for (int shift = 0; (nt >> shift) > 0; shift += 8, in ^= 1) {
        const uint32_t *kin = in ? a.keys[1] : a.keys[0], *vin = in ? a.vals[1] : a.vals[0];
        uint32_t *kout = in ? a.keys[0] : a.keys[1], *vout = in ? a.vals[0] : a.vals[1];
        base[tid] = 0;
        __syncthreads();
        for (int i = tid; i < n; i += kBlock) atomicAdd(&base[(kin[i] >> shift) & 255u], 1u);
        __syncthreads();
        const uint32_t cnt = base[tid], inc = wave_incl_scan(cnt);
        if (lane == 63) ws[w] = inc;
        __syncthreads();
        uint32_t pre = inc - cnt;
        for (int k = 0; k < w; k++) pre += ws[k];
        base[tid] = pre;
        for (int b = 0; b < n; b += kBlock) {
#pragma unroll
            for (int k = 0; k < kBlock / 64; k++) wcnt[k][tid] = 0;
            __syncthreads();
            const int i = b + tid;
            const bool valid = i < n;
            const uint32_t key = valid ? kin[i] : 0u, val = valid ? vin[i] : 0u, d = (key >> shift) & 255u;
            unsigned long long m = __ballot(valid);
#pragma unroll
            for (int bit = 0; bit < 8; bit++) {
                const bool on = (d >> bit) & 1u;
                const unsigned long long bb = __ballot(on);
                m &= on ? bb : ~bb;
            }
            const int rank = __popcll(m & lt);
            if (valid && rank == 0) wcnt[w][d] = (uint32_t)__popcll(m);
            __syncthreads();
            if (valid) {
                uint32_t p = base[d] + (uint32_t)rank;
                for (int k = 0; k < w; k++) p += wcnt[k][d];
                kout[p] = key;
                vout[p] = val;
            }
            __syncthreads();
            for (int k = 0; k < kBlock / 64; k++) base[tid] += wcnt[k][tid];
            __syncthreads();
        }
    }
    // tile offsets from the sorted keys: slot i begins the tiles after the previous slot's key
    const uint32_t* keys = in ? a.keys[1] : a.keys[0];
    for (int i = tid; i <= n; i += kBlock) {
        const int k = i < n ? (int)keys[i] : nt + 1, kp = i > 0 ? (int)keys[i - 1] : -1;
        for (int t = kp + 1; t <= k; t++) {
            a.toff[t] = i;
            if (t == nt) *a.n_live = i;
        }
    }
    if (tid == 0) atomicAdd(a.n_fallback, 1ull);
}

constexpr int kMigItems = 8;  // slots per thread per round of the scatter

// Workgroup s < n_tiles: the particles of source tile s (the newly dead go to the dead bin after
// the live ones); workgroup n_tiles: the offsets of the dead bin and the live count.
// A wave takes 64 x kMigItems consecutive slots of a round.  Nine in ten particles stay in their
// tile: their test is one AND and one compare of the packed cell, their rank a ballot and a count
// of bits.  The others go to a list in LDS, in slot order, and are given direction and rank 64 at a
// time, so that the long part runs on full waves.  Bound by memory, 8 bytes a particle: the two
// species of the 2048^2 leaky box (268M particles) take 0.49 ms together, 4.4 TB/s where a copy
// reaches 5.0 (0.71 ms with the ballots of the direction bits taken for every particle).
__device__ __attribute__((always_inline)) inline void mig_scatter_body(const MigArgs& a, int blk, int, int)
{
    const MigGeo& g = a.g;
    __shared__ uint32_t run[2][kMigDirs];               // next place per direction
    __shared__ uint32_t wc[kBlock / 64][kMigDirs];      // leaving particles per wave and direction
    __shared__ uint32_t wstay[kBlock / 64];             // staying particles per wave
    __shared__ uint32_t lcell[kBlock / 64][64 * kMigItems];   // the list: cell, then direction and rank
    __shared__ uint16_t lslot[kBlock / 64][64 * kMigItems];   // slot in the wave's range
    __shared__ uint32_t sl[kMigSmall + 1], ws[2][kBlock / 64];
    static_assert(sizeof(lcell) >= 4 * (256 * (1 + kBlock / 64) + kBlock / 64), "the lone sort's LDS");
    if (*a.fallback) {
        if (blk == 0) radix_alone(a, lcell[0]);
        return;
    }
    const int nt = g.n_tiles, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int s = blk == nt ? nt : xcd_contiguous(blk, nt);
    uint32_t live, dead_pre;
    const uint32_t* start = a.start;
    if (nt <= kMigSmall) {  // the scans here: 4 tiles a thread
        constexpr int kPer = kMigSmall / kBlock;
        uint32_t v[kPer], sum = 0, dsum = 0;
#pragma unroll
        for (int k = 0; k < kPer; k++) {
            const int t = tid * kPer + k;
            v[k] = t < nt ? a.tot[t] : 0u;
            dsum += t < s && t < nt ? a.dcnt[t] : 0u;
            sum += v[k];
        }
        const uint32_t inc = wave_incl_scan(sum);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) dsum += __shfl_xor(dsum, o, 64);
        if (lane == 63) {
            ws[0][w] = inc;
            ws[1][w] = dsum;
        }
        __syncthreads();
        uint32_t r = inc - sum;
        live = dead_pre = 0;
#pragma unroll
        for (int k = 0; k < kBlock / 64; k++) {
            if (k < w) r += ws[0][k];
            live += ws[0][k];
            dead_pre += ws[1][k];
        }
#pragma unroll
        for (int k = 0; k < kPer; k++) {
            sl[tid * kPer + k] = r;
            r += v[k];
        }
        __syncthreads();
        start = sl;
    } else {
        live = start[nt];
        dead_pre = a.dpre[s];
    }
    if (s == nt) {
        // the slots of the previous dead bin stay dead at the end; nothing reads the
        // permutation past the live count, so they are not enumerated again
        if (tid == 0) {
            a.toff[nt] = (int32_t)live;
            a.toff[nt + 1] = a.n_upper;
            *a.n_live = (int32_t)live;
        }
        return;
    }
    const int32_t* __restrict__ cell = a.cell;
    uint32_t* __restrict__ perm = a.which ? a.vals[1] : a.vals[0];
    int sx, sy, sz;
    tile_coords(g, s, sx, sy, sz);
    const int co = mig_center(g, sy, true), ci = mig_center(g, sy, false);
    if (tid == 0) a.toff[s] = (int32_t)start[s];
    if (tid < kMigDirs) {
        uint32_t b = 0;
        if (tid == kMigDead) {
            b = live + dead_pre;
        } else {
            int dx, dy, dz;
            dir_steps(tid, dx, dy, dz);
            if (dir_possible(g, dx, dy, dz))
                b = start[mig_dst(g, sx, sy, sz, dx, dy, dz)] + a.mpre[(size_t)s * kMigDirs + tid];
        }
        run[0][tid] = b;
    }
    // bits of the packed cell that name the tile (bit 31 too: set in a dead particle's cell)
    const uint32_t tmask = (a.cc.m0 >> g.lt[0] << g.lt[0]) | (a.cc.m1 >> g.lt[1] << g.lt[1] << a.cc.b0) |
                           (uint32_t)(0xFFFFFFFFull << (a.cc.b0 + a.cc.b1 + g.lt[2])) | 0x80000000u;
    const uint32_t tcode = (uint32_t)a.cc.encode(sx << g.lt[0], sy << g.lt[1], sz << g.lt[2]);
    const int beg = a.toff_prev[s], end = a.toff_prev[s + 1];
    int p = 0;
    for (int cb = beg; cb < end; cb += kBlock * kMigItems) {
        const int wb = cb + w * 64 * kMigItems + lane;
        uint32_t c[kMigItems];
        unsigned long long ms[kMigItems];
#pragma unroll
        for (int j = 0; j < kMigItems; j++) c[j] = wb + j * 64 < end ? (uint32_t)cell[wb + j * 64] : 0u;
        if (lane < kMigDirs) wc[w][lane] = 0u;
        int nl = 0, nst = 0;
#pragma unroll
        for (int j = 0; j < kMigItems; j++) {
            const bool valid = wb + j * 64 < end, stay = valid && (c[j] & tmask) == tcode;
            ms[j] = __ballot(stay);
            const unsigned long long ml = __ballot(valid && !stay);
            if (valid && !stay) {
                const int e = nl + __builtin_amdgcn_mbcnt_hi((uint32_t)(ml >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ml, 0u));
                lcell[w][e] = c[j];
                lslot[w][e] = (uint16_t)(j * 64 + lane);
            }
            nl += __popcll(ml);
            nst += __popcll(ms[j]);
        }
        __builtin_amdgcn_wave_barrier();
        for (int b = 0; b < nl; b += 64) {
            const int e = b + lane;
            const int d = e < nl ? mig_dir(g, a.cc, sx, sy, sz, co, ci, (int32_t)lcell[w][e]) : -1;
            // lanes with the same key (direction + 1, 5 bits; 0 = none): the AND over the key
            // bits of the ballot of that bit or of its complement
            const uint32_t key = (uint32_t)(d + 1);
            unsigned long long same = ~0ull;
#pragma unroll
            for (int bit = 0; bit < 5; bit++) {
                const unsigned long long m = __ballot((key >> bit) & 1u);
                same &= ((key >> bit) & 1u) ? m : ~m;
            }
            const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
            const uint32_t before = d >= 0 ? wc[w][d] : 0u;
            __builtin_amdgcn_wave_barrier();
            // the lowest lane of each group adds the group's count (same wave: in order)
            if (d >= 0 && rank == 0) wc[w][d] = before + (uint32_t)__popcll(same);
            if (e < nl) lcell[w][e] = d >= 0 ? (uint32_t)d << 16 | (before + rank) : 0xFFFFFFFFu;
            __builtin_amdgcn_wave_barrier();
        }
        if (lane == 0) wstay[w] = (uint32_t)nst;
        __syncthreads();
        uint32_t at = run[p][kMigStay];
#pragma unroll
        for (int k = 0; k < kBlock / 64; k++)
            if (k < w) at += wstay[k];
#pragma unroll
        for (int j = 0; j < kMigItems; j++) {
            if ((ms[j] >> lane) & 1ull)
                perm[at + __builtin_amdgcn_mbcnt_hi((uint32_t)(ms[j] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ms[j], 0u))] =
                    (uint32_t)(wb + j * 64);
            at += (uint32_t)__popcll(ms[j]);
        }
        for (int e = lane; e < nl; e += 64) {
            const uint32_t v = lcell[w][e];
            if (v == 0xFFFFFFFFu) continue;
            const int d = (int)(v >> 16);
            uint32_t pos = run[p][d] + (v & 0xFFFFu);
#pragma unroll
            for (int k = 0; k < kBlock / 64; k++)
                if (k < w) pos += wc[k][d];
            perm[pos] = (uint32_t)(cb + w * 64 * kMigItems + lslot[w][e]);
        }
        if (tid < kMigDirs) {
            uint32_t r = run[p][tid];
#pragma unroll
            for (int k = 0; k < kBlock / 64; k++) r += tid == kMigStay ? wstay[k] : wc[k][tid];
            run[p ^ 1][tid] = r;
        }
        __syncthreads();
        p ^= 1;
    }
}
PIC_BATCH_KERNEL(mig_scatter, MigArgs, kBlock)

// the species of one box side by side
#define PIC_PAIR_KERNEL(name, NT)                                            \
    __global__ __launch_bounds__(NT) void name##_pair(MigPair a)             \
    {                                                                        \
        name##_body(a.s[blockIdx.y], (int)blockIdx.x, (int)gridDim.x, 0);    \
    }
PIC_PAIR_KERNEL(mig_offsets, kBlock)
PIC_PAIR_KERNEL(mig_scan, kScanBlock)
PIC_PAIR_KERNEL(mig_scatter, kBlock)

hipError_t sort_batch(SortBatchKind k, const void* table, UnitMap m, int blocks, hipStream_t st)
{
    if (blocks <= 0) return hipSuccess;
    const MigArgs* t = static_cast<const MigArgs*>(table);
    switch (k) {
    case kBatchMigOffsets: mig_offsets_batch<<<blocks, kBlock, 0, st>>>(t, m); break;
    case kBatchMigScan: mig_scan_batch<<<blocks, kScanBlock, 0, st>>>(t, m); break;
    case kBatchMigScatter: mig_scatter_batch<<<blocks, kBlock, 0, st>>>(t, m); break;
    }
    return hipGetLastError();
}

int sort_result_buffer(const Tiles& tl) { return radix_passes(tl) & 1; }
unsigned mig_offset_blocks(int nt) { return (unsigned)((nt + kBlock / 64 - 1) / (kBlock / 64)); }
bool mig_needs_scan(int nt) { return nt > kMigSmall; }

size_t migrate_scratch_words(int n_tiles) { return scan_scratch_words((int64_t)n_tiles + 1); }

// The scans take one workgroup each up to this many tiles, twelve launches (three for each of two scans and
// species) beyond.  The whole sort of two sparse species on 8 x 8 tiles, us, one workgroup / launches: 4096 tiles
// 40 / 84, 16384 118 / 160, 32761 220 / 251, 65536 430 / 432, 90000 586 / 565, 160000 1028 / 947; beside the
// Maxwell step of the 256^3 shearing box (32768 tiles) and the 2048^2 leaky box (16384) a step takes as long either way.
constexpr int kScanAlone = 1 << 16;

hipError_t migrate_sort(const MigPair& a, int n_species, uint32_t* const* scratch, hipStream_t st)
{
    const int nt = a.s[0].g.n_tiles;
    const dim3 y1(1, (unsigned)n_species);
    mig_offsets_pair<<<dim3(mig_offset_blocks(nt), y1.y), kBlock, 0, st>>>(a);
    if (nt > kScanAlone) {
        for (int s = 0; s < n_species; s++) {
            hipError_t e = scan_exclusive(a.s[s].tot, a.s[s].start, nt + 1, scratch[s], st);
            if (e == hipSuccess) e = scan_exclusive(a.s[s].dcnt, a.s[s].dpre, nt + 1, scratch[s], st);
            if (e != hipSuccess) return e;
        }
    } else if (mig_needs_scan(nt)) {
        mig_scan_pair<<<dim3(2, y1.y), kScanBlock, 0, st>>>(a);
    }
    mig_scatter_pair<<<dim3(nt + 1, y1.y), kBlock, 0, st>>>(a);
    return hipGetLastError();
}

}  // namespace pic
