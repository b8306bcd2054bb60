// Forward MPM step kernels for gfx950 and their host launchers.
//
// One step (Sec. 2.2, update-stress-last), 3-D:
//   1. scan_once       tile counts -> tile offsets, active tiles; beside it the
//                      halo tiles, empty ones that particles' nodes reach (past
//                      131,072 tiles scan_reduce and scan_down)
//   2. sort_gather     each tile's particles found where the last step left them,
//                      ranked by cell and previous slot: the permutation and the
//                      cells' counts.  Where no step has laid out the state:
//                      bucket (scatter by tile) and sort
//   3. p2g             one tile per workgroup, lane = cell: P2G (eq:update_m,
//                      momentum with the APIC affine term of App. B, internal
//                      force from the stress cache) summed in registers, written
//                      out as the tile's partial block
//   4. grid            over active and halo tiles: sums the partial blocks
//                      covering each node in a fixed order; v = P/m + dt g, walls
//                      (Sec. 5.3 friction law).  No floating-point atomics: the
//                      step is deterministic
//   5. g2p             per active tile: LDS node block, velocity, APIC C, velocity
//                      gradient, position, then the constitutive update; writes
//                      the state in the new sorted order, counts the next keys
//                      and marks where particles change their tile
// In 2-D, 2 and 3 are one kernel (sort_p2g2), which up to 2048 tiles does 1 as
// well where a step has laid out the state, and 4 is done by g2p.
#pragma once

#include <hip/hip_runtime.h>

#include <math.h>

#include <algorithm>

#include "mpm_device.hpp"
#include "mpm_runtime.hpp"

namespace mpm {

template <int D> struct TileShape;
// TE: cells per edge, BE: block nodes per edge, NB: block nodes.
template <> struct TileShape<3> { static constexpr int TE = 4, BE = 6, NB = 216; };
template <> struct TileShape<2> { static constexpr int TE = 8, BE = 10, NB = 100; };

// How a block lies in LDS: row and plane stride, size, and the place of block
// node i.  DenseBlock: as in memory.  PaddedBlock (3-D): lanes are cells, at
// x + LY y + LZ z over a tile's 4^3; with 8 and 52 a binary64 access meets each
// pair of banks from exactly two lanes, where the dense 6 and 36 collide.
template <int D>
struct DenseBlock {
    static constexpr int LY = TileShape<D>::BE, LZ = LY * LY, LN = TileShape<D>::NB;
    static __device__ __forceinline__ int at(int i) { return i; }
};
struct PaddedBlock {
    static constexpr int LY = 8, LZ = 52, LN = 312;
    static __device__ __forceinline__ int at(int i) { return (i / 36) * LZ + (i / 6) % 6 * LY + i % 6; }
};

constexpr int kSortCap = 1024;   // particles per tile sorted in LDS (larger: in perm)
// threads of a 3-D P2G workgroup, one tile each: two waves that split the node
// values; with FLIP, whose node values double (momentum with and without the
// internal force), four
template <bool FL> constexpr int kP2GBlock = FL ? 256 : 128;
// threads of a G2P workgroup (3-D binary64: smaller groups, measured faster)
template <class T, int D> constexpr int kG2PBlock = sizeof(T) == 8 && D == 3 ? 128 : 256;
template <class T> constexpr int kG2PNarrow2 = sizeof(T) == 8 ? 128 : 256;   // 2-D, see kSortNarrow2
// G2P loads the next tile's node block while it works on the current one
// (binary64: measured faster; binary32: slower)
template <class T> constexpr bool kG2PPrefetch = sizeof(T) == 8;
constexpr int kGridBlock = 128;  // threads of a grid-update workgroup
constexpr int kHaloAt = 2;       // meta[kHaloAt]: halo tiles of the step (see Halo)
constexpr int kHaloSum = 8;      // where it gathers in the context's meta
constexpr int kScanOnce = 1024;  // threads of the one-launch scan
// Tiles up to which the scan is one launch whose workgroups each sum all
// earlier counts: latency, not bytes, bounds the scan, and that trip is shorter
// than a launch until the counts of the last workgroup's sum take as long.
// Two launches and one: 1,000 tiles 12.4 and 6.9 us, 20,480 14.3 and 7.8, 64,000
// 15.1 and 10.1, 131,072 15.5 and 13.0, 262,144 16.4 and 18.0, 512,000 21.4 and
// 28.5.  Cylinder (65 k tiles) 13.8 and 9.9, columns 14.5 and 7.9 (11.5 and 8.6
// with the halo list beside it).
constexpr int kScanOnceTiles = 131072;

// Particle data read once per step (G2P's old state; P2G's inputs where the
// state outgrows the caches, see p2g_hint) and the part of G2P's output that no
// later kernel of the step reads (F or J, pid) go through the non-temporal
// cache hint.  Measured on the 3-D cylinder: G2P 140 -> 137 us binary32, 256 ->
// 246 binary64; the hint on the stores that P2G reads next (x, v, C, the stress
// cache) made G2P slower, so those stay ordinary stores.
template <class T>
__device__ __forceinline__ T ld_once(const T* p)
{
    return __builtin_nontemporal_load(p);
}
template <class T>
__device__ __forceinline__ void st_late(T v, T* p)
{
    __builtin_nontemporal_store(v, p);
}

// Active-list entry handled by this workgroup on iteration `it`.  Workgroup b
// runs on XCD b % 8; each XCD gets one contiguous chunk of the active list so
// that neighbouring tiles share that XCD's L2.
__device__ __forceinline__ int tile_entry(int it, int n_active)
{
    int nx = 8;
    int per = gridDim.x / nx;
    int xcd = blockIdx.x % nx;
    int lb = blockIdx.x / nx;
    int chunk = (n_active + nx - 1) / nx;
    int e = xcd * chunk + lb + it * per;
    int end = min((xcd + 1) * chunk, n_active);
    return e < end ? e : -1;
}

// Lane q: the active slot of neighbour q of a 3-D tile (x fastest, the tile
// itself at 13), -1 where that is empty or outside the grid or q > 26.
__device__ __forceinline__ int around_slot(const Geo& g, int tile, const int* __restrict__ tile_slot)
{
    const int lane = threadIdx.x & 63;
    int tc[3];
    tile_coords(g, tile, tc);
    const int tx = tc[0] + lane % 3 - 1, ty = tc[1] + (lane / 3) % 3 - 1, tz = tc[2] + lane / 9 - 1;
    if (lane > 26 || tx < 0 || ty < 0 || tz < 0 || tx >= g.ntile[0] || ty >= g.ntile[1] || tz >= g.ntile[2]) return -1;
    return tile_slot[(tz * g.ntile[1] + ty) * g.ntile[0] + tx];
}

// Tile handled by this wave (one of the workgroup's NW) on iteration `it`: an
// active tile, then a halo tile, each list in one contiguous chunk per
// XCD; -1: none left.
template <int NW>
__device__ __forceinline__ int node_tile(int it, const int* __restrict__ meta, const ActiveTile* __restrict__ active, int ntiles)
{
    const int n_active = meta[0], n_halo = meta[kHaloAt];
    const int xcd = blockIdx.x % 8;
    int i = ((int)(blockIdx.x / 8) + it * (int)(gridDim.x / 8)) * NW + (int)(threadIdx.x >> 6);
    const int ca = (n_active + 7) / 8, ch = (n_halo + 7) / 8;
    const int na = max(min((xcd + 1) * ca, n_active) - xcd * ca, 0), nh = max(min((xcd + 1) * ch, n_halo) - xcd * ch, 0);
    if (i < na) return active[xcd * ca + i].tile;
    i -= na;
    return i < nh ? active[ntiles - 1 - (xcd * ch + i)].tile : -1;
}

// ---------------------------------------------------------------------------
// Block-wide exclusive scan of two ints (256 threads).
// ---------------------------------------------------------------------------

__device__ __forceinline__ void block_scan2(int a, int b, int& ex_a, int& ex_b, int& tot_a, int& tot_b)
{
    __shared__ int sa[4], sb[4];
    int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int ia = a, ib = b;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        int ta = __shfl_up(ia, o), tb = __shfl_up(ib, o);
        if (lane >= o) { ia += ta; ib += tb; }
    }
    if (lane == 63) { sa[w] = ia; sb[w] = ib; }
    __syncthreads();
    int pa = 0, pb = 0;
    for (int k = 0; k < w; ++k) { pa += sa[k]; pb += sb[k]; }
    tot_a = sa[0] + sa[1] + sa[2] + sa[3];
    tot_b = sb[0] + sb[1] + sb[2] + sb[3];
    ex_a = pa + ia - a;
    ex_b = pb + ib - b;
    __syncthreads();
}

// Halo tiles (3-D): the empty ones that a particle's block of nodes can reach,
// that is, with particles in one of the seven tiles below.  The grid kernels
// visit them after the active tiles.  They are appended to `active` from its
// end, in no particular order (no result depends on it); their number gathers in
// `n`, which the step's sort moves to meta[kHaloAt] and clears.  Workgroups of
// the scan's launch beside those that scan form the list, so that it is done
// when they are: as work of the scanning ones it took 3.5 us more, in the sort 5
// (its wave waits for the list's counter), in P2G 7 (it costs the stream
// registers).
struct Halo {
    int* n;        // nullptr: no list (2-D)
    int nx, ny;    // tiles along x and y
    int first;     // the launch's first workgroup that forms the list
};
__device__ __forceinline__ void halo_list(const Halo& h, const int* __restrict__ count, int ntiles, ActiveTile* __restrict__ active)
{
    for (int t = ((int)blockIdx.x - h.first) * (int)blockDim.x + (int)threadIdx.x; t - (int)(threadIdx.x & 63) < ntiles;
         t += ((int)gridDim.x - h.first) * (int)blockDim.x) {
        const int tx = t % h.nx, ty = (t / h.nx) % h.ny, tz = t / (h.nx * h.ny);
        int own = 1, below = 0;
        if (t < ntiles) {
            own = count[t];
#pragma unroll
            for (int m = 1; m < 8; ++m) {
                const int bx = m & 1, by = (m >> 1) & 1, bz = m >> 2;
                if (tx >= bx && ty >= by && tz >= bz) below |= count[t - bx - h.nx * (by + h.ny * bz)];
            }
        }
        const bool is = own == 0 && below != 0;
        const unsigned long long m = __ballot(is);
        if (!m) continue;
        const int lane = threadIdx.x & 63;
        int at = 0;   // one atomic per wave
        if (lane == 0) at = atomicAdd(h.n, __popcll(m));
        at = __builtin_amdgcn_readfirstlane(at) + __popcll(m & ((1ull << lane) - 1ull));
        if (is) active[ntiles - 1 - at].tile = t;
    }
}
// At the start of a step's sort, one thread.
__device__ __forceinline__ void halo_take(int* __restrict__ n, int* __restrict__ meta)
{
    meta[kHaloAt] = *n;
    *n = 0;
}

// Particles that left their tile's neighbourhood in a step (beyond the CFL
// limit), which the next step's sort does not meet in the ranges around their new
// tile: chained per new tile by G2P, in no order, through their slots.  One array:
// the marks of the neighbours, `moved`, each tile's first slot or -1, and per slot
// the next.
struct Far {
    int* moved;
    int ntiles;
    __device__ __forceinline__ int& head(int tile) const { return moved[(long long)ntiles + tile]; }
    __device__ __forceinline__ int& next(int slot) const { return moved[2ll * ntiles + slot]; }
    __device__ __forceinline__ void push(int tile, int slot) const { next(slot) = atomicExch(&head(tile), slot); }
};
constexpr int kFarBit = 1 << 27;   // of `moved` (3-D): the tile has such a chain
// A tile of more particles than this goes through all keys instead of its chain,
// which is a serial walk, and ranked by counting: at most 4096 tiles are.
constexpr int kFarCrowd = 4096;
__device__ __forceinline__ bool far_scans_all(int cnt, long long N) { return cnt > kFarCrowd && cnt > N / 4096; }

// What the scan leaves for tile t with c particles from `off` on; slot: its
// place in the active list.
__device__ __forceinline__ void scan_put(int t, int c, int off, int& slot, int* __restrict__ tile_off,
                                         int* __restrict__ tile_slot, ActiveTile* __restrict__ active,
                                         int2* __restrict__ range, int* __restrict__ count_next)
{
    tile_off[t] = off;
    if (range) range[t] = make_int2(off, c);
    if (count_next) count_next[t] = 0;
    if (c > 0) {
        tile_slot[t] = slot;
        ActiveTile e;
        e.tile = t;
        e.off = off;
        e.cnt = c;
        e.pad = 0;
        active[slot] = e;
        ++slot;
    } else {
        tile_slot[t] = -1;
    }
}

// The scan in one launch: each workgroup sums all earlier counts itself, 32 per
// thread and trip.
template <int Unused = 0>
__global__ __launch_bounds__(kScanOnce) void k_scan_once(const int* __restrict__ count, int ntiles,
                                                         int* __restrict__ tile_off, int* __restrict__ tile_slot,
                                                         ActiveTile* __restrict__ active, int* __restrict__ meta,
                                                         int2* __restrict__ range, int* __restrict__ count_next, Halo halo)
{
    constexpr int PER = kScanChunk / kScanOnce, NW = kScanOnce / 64, BATCH = 8;
    __shared__ int s_sum[NW][4];
    if ((int)blockIdx.x >= halo.first) {
        halo_list(halo, count, ntiles, active);
        return;
    }
    const int base = blockIdx.x * kScanChunk, t0 = base + (int)threadIdx.x * PER;
    int c[PER], ls = 0, la = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        c[k] = t0 + k < ntiles ? count[t0 + k] : 0;
        ls += c[k];
        la += c[k] > 0;
    }
    const int4* before = (const int4*)count;   // base is a multiple of 4
    int ps = 0, pa = 0;
    for (int i0 = 0; i0 < base / 4; i0 += BATCH * kScanOnce) {
        int4 v[BATCH];
#pragma unroll
        for (int q = 0; q < BATCH; ++q) {
            const int i = i0 + q * kScanOnce + (int)threadIdx.x;
            v[q] = i < base / 4 ? before[i] : make_int4(0, 0, 0, 0);
        }
#pragma unroll
        for (int q = 0; q < BATCH; ++q) {
            ps += v[q].x + v[q].y + v[q].z + v[q].w;
            pa += (v[q].x > 0) + (v[q].y > 0) + (v[q].z > 0) + (v[q].w > 0);
        }
    }
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int is = ls, ia = la;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int ts = __shfl_up(is, o), ta = __shfl_up(ia, o);
        if (lane >= o) { is += ts; ia += ta; }
        ps += __shfl_xor(ps, o);
        pa += __shfl_xor(pa, o);
    }
    if (lane == 63) {
        s_sum[w][0] = ps;
        s_sum[w][1] = pa;
        s_sum[w][2] = is;
        s_sum[w][3] = ia;
    }
    __syncthreads();
    int off = is - ls, slot = ia - la;
    for (int k = 0; k < NW; ++k) {
        off += s_sum[k][0] + (k < w ? s_sum[k][2] : 0);
        slot += s_sum[k][1] + (k < w ? s_sum[k][3] : 0);
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        if (t0 + k < ntiles) scan_put(t0 + k, c[k], off, slot, tile_off, tile_slot, active, range, count_next);
        off += c[k];
    }
    if ((int)blockIdx.x == halo.first - 1 && threadIdx.x == kScanOnce - 1) {
        meta[0] = slot;
        meta[1] = off;
    }
}

template <int Unused = 0>
__global__ __launch_bounds__(kBlock) void k_scan_reduce(const int* __restrict__ count, int ntiles,
                                                        int* __restrict__ part)
{
    int base = blockIdx.x * kScanChunk;
    int s = 0, a = 0;
    for (int i = threadIdx.x; i < kScanChunk; i += kBlock) {
        int t = base + i;
        if (t < ntiles) {
            int c = count[t];
            s += c;
            a += (c > 0);
        }
    }
    int es, ea, ts, ta;
    block_scan2(s, a, es, ea, ts, ta);
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = ts;
        part[2 * blockIdx.x + 1] = ta;
    }
}

template <int Unused = 0>
__global__ __launch_bounds__(kBlock) void k_scan_down(const int* __restrict__ count, int ntiles,
                                                      const int* __restrict__ part,
                                                      int* __restrict__ tile_off, int* __restrict__ tile_slot,
                                                      ActiveTile* __restrict__ active, int* __restrict__ meta,
                                                     int2* __restrict__ range, int* __restrict__ count_next, Halo halo)
{
    if ((int)blockIdx.x >= halo.first) {
        halo_list(halo, count, ntiles, active);
        return;
    }
    // prefix of the earlier chunks
    int ps = 0, pa = 0;
    for (int i = threadIdx.x; i < (int)blockIdx.x; i += kBlock) {
        ps += part[2 * i];
        pa += part[2 * i + 1];
    }
    int e0, e1, base_s, base_a;
    block_scan2(ps, pa, e0, e1, base_s, base_a);
    constexpr int PER = kScanChunk / kBlock;
    int t0 = blockIdx.x * kScanChunk + threadIdx.x * PER;
    int c[PER];
    int ls = 0, la = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        int t = t0 + k;
        c[k] = (t < ntiles) ? count[t] : 0;
        ls += c[k];
        la += (c[k] > 0);
    }
    int ex_s, ex_a, tot_s, tot_a;
    block_scan2(ls, la, ex_s, ex_a, tot_s, tot_a);
    int off = base_s + ex_s, slot = base_a + ex_a;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        int t = t0 + k;
        if (t < ntiles) scan_put(t, c[k], off, slot, tile_off, tile_slot, active, range, count_next);
        off += c[k];
    }
    if ((int)blockIdx.x == halo.first - 1 && threadIdx.x == kBlock - 1) {
        meta[0] = slot;
        meta[1] = off;
    }
}

// Scatter every particle into its tile's range (order inside a tile is
// arbitrary here; k_sort, in 2-D k_sort_p2g2, ranks them).  Leaves count[] at zero.  A
// thread takes kBucketPer particles, kBlock apart, whose loads, range
// reservations and stores are each issued together.
constexpr int kBucketPer = 4;

template <int Unused = 0>
__global__ __launch_bounds__(kBlock) void k_bucket(long long N, const int* __restrict__ key,
                                                   int* __restrict__ count, const int* __restrict__ tile_off,
                                                   int* __restrict__ tmp, int* __restrict__ tmpk)
{
    const long long j0 = (long long)blockIdx.x * (kBlock * kBucketPer) + threadIdx.x;
    int k[kBucketPer], head[kBucketPer], len[kBucketPer], rank[kBucketPer], base[kBucketPer];
#pragma unroll
    for (int q = 0; q < kBucketPer; ++q) {
        const long long j = j0 + q * kBlock;
        k[q] = j < N ? key[j] : -1;
    }
#pragma unroll
    for (int q = 0; q < kBucketPer; ++q) {
        const bool valid = j0 + q * kBlock < N;
        wave_runs(valid ? (k[q] >> 6) : -1, valid, head[q], len[q], rank[q]);
        base[q] = 0;
        if (valid && rank[q] == 0) base[q] = atomicSub(&count[k[q] >> 6], len[q]) - len[q];
    }
#pragma unroll
    for (int q = 0; q < kBucketPer; ++q) {
        const long long j = j0 + q * kBlock;
        const int b = __shfl(base[q], head[q]);
        if (j < N) {
            const int slot = tile_off[k[q] >> 6] + b + rank[q];
            tmp[slot] = (int)j;
            tmpk[slot] = k[q];
        }
    }
}

// A new state in one launch (copies, fills and keys were eight to eleven, each a
// launch's latency: initial state, 20 steps and reads of 8,192 particles 300 ->
// 285 us, of 32,768 in binary64 433 -> 418): x and v of
// N particles (component-major), everything else zero up to the capacity, the
// slots' particles in order, keys and tile counts (cleared before, clear_keys).
template <class T, int D>
__global__ __launch_bounds__(kBlock) void k_init(Geo g, Phys<T> P, const T* __restrict__ x, const T* __restrict__ v, long long N,
                                                 PView<T> s, int nsc, T* __restrict__ eps0, T* __restrict__ eps1,
                                                 int* __restrict__ key, int* __restrict__ count)
{
    const long long j = (long long)blockIdx.x * kBlock + threadIdx.x;
    const bool valid = j < N;
    int k = 0;
    if (valid) {
        T xp[D];
#pragma unroll
        for (int a = 0; a < D; ++a) {
            xp[a] = x[a * N + j];
            s.x[a * s.cap + j] = xp[a];
            s.v[a * s.cap + j] = v[a * N + j];
        }
        s.pid[j] = (int32_t)j;
        k = cell_key<T, D>(g, xp, P.inv);
        key[j] = k;
    }
    if (j < s.cap) {
        // C, G (or dJ) and S follow v contiguously
        for (int q = 0; q < nsc - 2 * D; ++q) s.C[q * s.cap + j] = T(0);
        if (eps0) eps0[j] = T(0);
        if (eps1) eps1[j] = T(0);
    }
    int head, len, rank;
    wave_runs(valid ? (k >> 6) : -1, valid, head, len, rank);
    if (valid && rank == 0) atomicAdd(&count[k >> 6], len);
}

// The tiles' counts and the marks of the last step's moves to none.
template <int Unused = 0>
__global__ __launch_bounds__(kBlock) void k_clear_keys(int* __restrict__ count, Far far, int ntiles)
{
    for (int t = blockIdx.x * kBlock + threadIdx.x; t < ntiles; t += gridDim.x * kBlock) {
        count[t] = 0;
        if (far.moved) {
            far.moved[t] = 0;
            far.head(t) = -1;
        }
    }
}

// The layout of the current state from one set of ranges (2-D: and counts) to
// the other.
template <int Unused = 0>
__global__ __launch_bounds__(kBlock) void k_copy_layout(const int2* __restrict__ range, int2* __restrict__ range_to,
                                                        const int* __restrict__ count, int* __restrict__ count_to, int ntiles)
{
    for (int t = blockIdx.x * kBlock + threadIdx.x; t < ntiles; t += gridDim.x * kBlock) {
        range_to[t] = range[t];
        if (count) count_to[t] = count[t];
    }
}

template <class T, int D>
__global__ __launch_bounds__(kBlock) void k_keys(Geo g, Phys<T> P, PView<T> cur, long long N,
                                                 int* __restrict__ key, int* __restrict__ count)
{
    long long j = (long long)blockIdx.x * kBlock + threadIdx.x;
    bool valid = j < N;

    int k = 0;
    if (valid) {
        T xp[D];
#pragma unroll
        for (int a = 0; a < D; ++a) xp[a] = cur.x[a * cur.cap + j];
        k = cell_key<T, D>(g, xp, P.inv);
        key[j] = k;
    }
    int head, len, rank;
    wave_runs(valid ? (k >> 6) : -1, valid, head, len, rank);
    if (valid && rank == 0) atomicAdd(&count[k >> 6], len);
}

// ---------------------------------------------------------------------------
// P2G
// ---------------------------------------------------------------------------

template <class T>
__device__ __forceinline__ void weights_from_f(T f, T inv, T w[3], T dw[3])
{
    T a0 = T(1.5) - f, a1 = f - T(1), a2 = f - T(0.5);
    w[0] = T(0.5) * a0 * a0;
    w[1] = T(0.75) - a1 * a1;
    w[2] = T(0.5) * a2 * a2;
    dw[0] = -a0 * inv;
    dw[1] = T(-2) * a1 * inv;
    dw[2] = a2 * inv;
}

// Orders this wave's LDS accesses: the compiler may not move LDS reads or
// writes across it, and the hardware executes one wave's LDS operations in
// order, so a lane sees what another lane of the same wave wrote before.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The state of one particle that P2G reads for the momentum components
// [A0, A1): the position, those components of v, those rows of C and the
// stress cache.
template <class T, int D, int MAT, int A0 = 0, int A1 = D, bool NTL = true>
struct P2GIn {
    static constexpr int NS = mat_iso_stress(MAT) ? 1 : D * (D + 1) / 2;
    static constexpr int NA = A1 - A0;
    T x[D], v[NA], C[NA * D], S[NS];
    static __device__ __forceinline__ T ld(const T* p) { return NTL ? ld_once(p) : *p; }
    // Both waves of a tile read the position: in binary32 it is loaded without
    // the hint, so that the second wave finds it in the cache (cylinder 74.6 ->
    // 71.8 us, G2P 135.8 -> 134.7).  Binary64 keeps the hint (145.1 and 146.1,
    // G2P 252 and 256), and so does the stress (72.6; binary64 156).
    static constexpr bool kLdX = sizeof(T) == 4;
    __device__ __forceinline__ void load(const PView<T>& cur, int j)
    {
        const long long cap = cur.cap;
#pragma unroll
        for (int a = 0; a < D; ++a) x[a] = kLdX ? cur.x[a * cap + j] : ld(&cur.x[a * cap + j]);
#pragma unroll
        for (int a = 0; a < NA; ++a) v[a] = ld(&cur.v[(A0 + a) * cap + j]);
#pragma unroll
        for (int q = 0; q < NA * D; ++q) C[q] = ld(&cur.C[(A0 * D + q) * cap + j]);
#pragma unroll
        for (int q = 0; q < NS; ++q) S[q] = ld(&cur.S[q * cap + j]);
    }
};

// Index of entry (a, b) in the packed symmetric storage of the stress cache
// (3-D: 00 11 22 01 02 12; 2-D: 00 11 01).
template <int D>
__host__ __device__ constexpr int sym_index(int a, int b)
{
    return a == b ? a : (D == 2 ? 2 : (a + b == 1 ? 3 : (a + b == 2 ? 4 : 5)));
}

// One particle's P2G contribution (eq:update_m, the momentum with the APIC
// affine term of App. B, and the internal force -dt V_p sigma_p grad phi) in
// the momentum components [A0, A1).  Weights, x_i - x_p and grad phi factor over
// the axes, and so do the affine term and the force of each axis: with
//   E^b_a(k) = (w dd)_b(k) m C_ab + dw_b(k) fs_ab,  fs = -dt V_p sigma_p,
// the value at node (kx, ky, kz) is
//   P_a = w_x w_y w_z m v_a + E^x_a w_y w_z + w_x E^y_a w_z + w_x w_y E^z_a
//       = w_x U_a + (w_y w_z) E^x_a,
//   U_a = w_z (w_y m v_a + E^y_a) + w_y E^z_a  (2-D: without the z factors),
// two multiply-adds per node and two per line along x: 93 per component, where
// one term each for velocity, affine part and force per node was 144.
// Without FORCE (FLIP's v_i^n) fs = 0.  For each of the 3^D stencil nodes,
// sink(k, n, wx, mw, wyz, U, Ex) receives the offset index k, the node's index n
// in the tile's LDS block, the factors of the mass w_x mw and of P_a = w_x U_a +
// wyz Ex_a.
template <class T, int D, int MAT, int A0, int A1, bool FORCE, bool NTL, class Sink>
__device__ __forceinline__ void p2g_particle(const Phys<T>& P, const P2GIn<T, D, MAT, A0, A1, NTL>& in, const int lb[3],
                                             const int gb[3], Sink&& sink)
{
    constexpr int BE = TileShape<D>::BE, NA = A1 - A0;
    T w[D][3], dw[D][3], wd[D][3];
#pragma unroll
    for (int a = 0; a < D; ++a) {
        T x = in.x[a];
        T t = mul_exact(x, P.inv);
        T f = t - T(gb[a]);
        weights_from_f(f, P.inv, w[a], dw[a]);
#pragma unroll
        for (int k = 0; k < 3; ++k) wd[a][k] = w[a][k] * ((T(k) - f) * P.h);
    }
    // rows A0..A1-1 of m v and of the axis terms
    T mv[NA], E[D][3][NA];
#pragma unroll
    for (int a = 0; a < NA; ++a) {
        mv[a] = P.mass * in.v[a];
#pragma unroll
        for (int b = 0; b < D; ++b) {
            const T mC = P.mass * in.C[a * D + b];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                E[b][k][a] = wd[b][k] * mC;
                if constexpr (!FORCE) continue;
                if (mat_iso_stress(MAT)) {
                    if (A0 + a == b) E[b][k][a] = fma(dw[b][k], -P.dt * in.S[0], E[b][k][a]);
                } else {
                    E[b][k][a] = fma(dw[b][k], -P.dt * in.S[mat_iso_stress(MAT) ? 0 : sym_index<D>(A0 + a, b)], E[b][k][a]);
                }
            }
        }
    }
    // along y
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int a = 0; a < NA; ++a) E[1][k][a] = fma(w[1][k], mv[a], E[1][k][a]);
    constexpr int KZ = (D == 3) ? 3 : 1;
#pragma unroll
    for (int kz = 0; kz < KZ; ++kz) {
#pragma unroll
        for (int ky = 0; ky < 3; ++ky) {
            T wyz = w[1][ky], U[NA];
            if constexpr (D == 3) wyz *= w[D - 1][kz];
#pragma unroll
            for (int a = 0; a < NA; ++a) {
                U[a] = E[1][ky][a];
                if constexpr (D == 3) U[a] = fma(w[D - 1][kz], U[a], w[1][ky] * E[D - 1][kz][a]);
            }
            const T mw = P.mass * wyz;
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) {
                int n;
                if constexpr (D == 3) n = ((lb[2] + kz) * BE + lb[1] + ky) * BE + lb[0] + kx;
                else n = (lb[1] + ky) * BE + lb[0] + kx;
                sink((kz * 3 + ky) * 3 + kx, n, w[0][kx], mw, wyz, U, E[0][kx]);
            }
        }
    }
}

// Node index in the tile's LDS block of stencil offset k for a lane whose
// cell sits at lb.
template <int D>
__device__ __forceinline__ int block_node(const int lb[3], int k)
{
    constexpr int BE = TileShape<D>::BE;
    int kx = k % 3, ky = (k / 3) % 3, kz = k / 9;
    if constexpr (D == 3) return ((lb[2] + kz) * BE + lb[1] + ky) * BE + lb[0] + kx;
    else return (lb[1] + ky) * BE + lb[0] + kx;
}

// Position inside its tile of the particle of rank q in cell c, for the
// order (rank, cell): all cells' rank-0 particles first, then rank 1, ...
//   pos = sum_c' min(cnt[c'], q) + #{c' < c : cnt[c'] > q}.
// For q < 64 the two sums come from a table (the cells with more than q
// particles as a 64-bit mask, and the running count of earlier ranks);
// deeper ranks, which only crowded cells reach, count directly.
__device__ __forceinline__ int rank_major_pos(int c, int q, const unsigned long long* rmask, const int* roff,
                                              const int* cnt)
{
    if (q < 64) return roff[q] + __popcll(rmask[q] & ((1ull << c) - 1ull));
    // read through volatile: keeps the compiler from hoisting the 64 counts
    // into registers out of the callers' particle loops
    const volatile int* vc = cnt;
    int r = 0;
#pragma unroll 1
    for (int c2 = 0; c2 < 64; ++c2) {
        int n = vc[c2];
        r += min(n, q) + ((c2 < c && n > q) ? 1 : 0);
    }
    return r;
}

// ---------------------------------------------------------------------------
// Sort inside a tile: by rank within the cell (previous slot order), then by
// cell, so that the r-th particles of the 64 cells are adjacent in memory
// ---------------------------------------------------------------------------

struct TileSort {
    int cnt[64], off[64], cur[64], roff[64];
    unsigned long long rmask[64];
    int unord[kSortCap], sorted[kSortCap];
    unsigned char ucell[kSortCap];
    int found;
};

// One wave: from the histogram cnt the cells' offsets, the number of particles
// found and the rank table (cells with more than q particles, and the count of
// earlier ranks).
__device__ __forceinline__ void tile_sort_scan(TileSort& s, int lane)
{
    const int v = s.cnt[lane];
    int inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(inc, o);
        if (lane >= o) inc += t;
    }
    s.off[lane] = inc - v;
    if (lane == 63) s.found = inc;
    int run = 0;
    for (int q = 0; q < 64; ++q) {
        const unsigned long long m = __ballot(v > q);
        if (!m) break;
        if (lane == 0) {
            s.rmask[q] = m;
            s.roff[q] = run;
        }
        run += __popcll(m);
    }
}

// Notes the particle of slot j in its cell's range (arbitrary order inside):
// in LDS, or for a crowded tile in the tile's range of perm.
__device__ __forceinline__ void tile_sort_place(TileSort& s, bool in_lds, int c, int j, int* __restrict__ perm_tile)
{
    const int u = s.off[c] + atomicAdd(&s.cur[c], 1);
    if (in_lds) {
        s.unord[u] = j;
        s.ucell[u] = (unsigned char)c;
    } else {
        perm_tile[u] = j;
    }
}

// Ranks the placed particles inside their cells by previous slot and writes
// the tile's range of perm.  Tiles of up to kSortCap particles in LDS (s.sorted
// holds the order afterwards); crowded tiles stage the result in their range of
// tmp, whose bucketed entries are no longer needed.
template <int NT>
__device__ __forceinline__ void tile_sort_finish(TileSort& s, bool in_lds, int cnt, int* __restrict__ perm_tile,
                                                 int* __restrict__ tmp_tile)
{
    const int tid = threadIdx.x;
    if (in_lds) {
        __syncthreads();
        for (int u = tid; u < cnt; u += NT) {
            const int c = s.ucell[u], j = s.unord[u];
            const int o = s.off[c], n = s.cnt[c], last = o + n - 1;
            int rank = 0;
            // four independent LDS reads per pass; reads past the cell's range
            // repeat its last entry and are not counted
            for (int q = 0; q < n; q += 4) {
                int e[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) e[i] = s.unord[min(o + q + i, last)];
#pragma unroll
                for (int i = 0; i < 4; ++i) rank += (q + i < n && e[i] < j) ? 1 : 0;
            }
            s.sorted[rank_major_pos(c, rank, s.rmask, s.roff, s.cnt)] = j;
        }
        __syncthreads();
        for (int k = tid; k < cnt; k += NT) perm_tile[k] = s.sorted[k];
    } else {
        __threadfence_block();
        __syncthreads();
        for (int k = tid; k < cnt; k += NT) {
            int lo = 0;
#pragma unroll
            for (int step = 32; step >= 1; step >>= 1)
                if (lo + step < 64 && s.off[lo + step] <= k) lo += step;
            const int j = perm_tile[k], o = s.off[lo], n = s.cnt[lo];
            int rank = 0;
            for (int q = 0; q < n; ++q) rank += perm_tile[o + q] < j;
            tmp_tile[rank_major_pos(lo, rank, s.rmask, s.roff, s.cnt)] = j;
        }
        __threadfence_block();
        __syncthreads();
        const volatile int* rm = tmp_tile;
        for (int k = tid; k < cnt; k += NT) perm_tile[k] = rm[k];
        __threadfence_block();
        __syncthreads();
    }
}

// The previous step's layout and this step's, for kernels that gather.
struct Ranges {
    int* count;              // particles per tile, by the current keys
    int* count_next;         // 2-D: cleared for this step's G2P (3-D: count itself is)
    const int2* range;       // previous sort: first slot and number of each tile's particles
    int2* range_next;        // this sort
    int* moved;              // 3-D: bit per neighbour that particles came from, kFarBit (cleared for this step's G2P);
                             // the chains of the last step behind it (see Far; left empty for this step's G2P)
    const int* key;
    const int* tile_key;     // 2-D: the first kTileRow keys of every tile's range, a row per tile
    int* tile_perm;          // 2-D: the same of perm (null: not kept)
    long long N;
};

// 3-D: sorts each tile's particles into perm and keeps the cells' counts for
// P2G, in a kernel of its own: the sort is a chain of round trips that needs few
// registers, P2G a stream that fills them.
//
// Where the previous step's layout is known, the particles are found where that
// step left them, without the scatter over the grid.  G2P left those of each
// tile in one range of slots, their new keys beside them, and set a bit of the
// destination's word for every neighbour that one came from; a tile reads the
// keys of its own range and of the few ranges marked.  Ranges follow the order
// of the tiles, so taken in that order the particles come by ascending slot, and
// a particle's rank is the number already seen in its cell: one wave per tile
// counts along, 64 keys at a time (lanes of one cell are found by six ballots),
// and no wave waits for another.  A step moves a particle to a neighbouring tile
// at most; those that moved further (a step beyond the CFL limit) are chained to
// their new tile (see Far), sorted by slot and taken between the ranges, so that
// such a step costs each particle a few trips to memory, too: with all of 2.65 M
// particles moved 20 cells the step after takes 0.89 ms (0.26 without), where
// every tile went through all keys 5.9, and more with every tile and particle.
// Cylinder, 2,780,000 particles: 20 us between events, where the scatter took 13
// and the sort, by LDS placement inside P2G at its three waves per SIMD, about 25
// of P2G's 94 (binary32; 19 in a kernel of its own); 29 once the sand moves and
// tiles hold more than 512.  A wave is one chain: four dependent trips to memory
// and one more for each range marked, the counting of eight batches, the rank
// table and the placement.
constexpr int kSortBlock = 256;
constexpr int kOwnBatches = 8;   // batches of a tile's own range held in registers (512 particles, 8 per cell)

// One wave: takes a tile's chain and leaves its slots, ascending, in the end of
// the tile's range of tmp; their number (0 also for a crowded tile).
__device__ __forceinline__ int far_sorted(const Far& far, long long N, const ActiveTile& at, int* __restrict__ tmp,
                                          int* __restrict__ scratch)
{
    const int lane = threadIdx.x & 63;
    int j = __builtin_amdgcn_readfirstlane(far.head(at.tile)), n = 0;
    if (far_scans_all(at.cnt, N)) j = -1;
    for (; j >= 0 && n < at.cnt; ++n) {
        if (lane == 0) scratch[n] = j;
        j = __builtin_amdgcn_readfirstlane(far.next(j));
    }
    if (lane == 0) far.head(at.tile) = -1;
    __threadfence_block();
    for (int u = lane; u < n; u += 64) {
        const int f = scratch[u];
        int r = 0;
        for (int q = 0; q < n; ++q) r += scratch[q] < f;
        tmp[at.off + at.cnt - n + r] = f;
    }
    __threadfence_block();
    return n;
}

template <int Unused = 0>
__global__ __launch_bounds__(kSortBlock) __attribute__((amdgpu_waves_per_eu(8))) void k_sort_gather(Geo g, Ranges rg, int* __restrict__ meta, int* __restrict__ n_halo,
                                                            const ActiveTile* __restrict__ active, int* __restrict__ tmp,
                                                            int* __restrict__ tmpk, int* __restrict__ perm,
                                                            int* __restrict__ cell_cnt)
{
    constexpr int NW = kSortBlock / 64;
    __shared__ int s_cnt[NW][64], s_roff[NW][64];
    __shared__ unsigned long long s_rmask[NW][64];
    const int n_active = meta[0];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const unsigned long long below = (1ull << lane) - 1ull;
    int* cnt = s_cnt[w];
    if (blockIdx.x == 0 && threadIdx.x == 0) halo_take(n_halo, meta);
    // entries by wave: one contiguous chunk of the active list per XCD
    const int chunk = (n_active + 7) / 8, xcd = blockIdx.x % 8, per = (int)(gridDim.x / 8) * NW;
    const int end = min((xcd + 1) * chunk, n_active);
    for (int e = xcd * chunk + (int)(blockIdx.x / 8) * NW + w; e < end; e += per) {
        const ActiveTile at = active[e];
        const int2 own = rg.range[at.tile];
        const unsigned from = (unsigned)__builtin_amdgcn_readfirstlane(rg.moved[at.tile]);   // the wave's one tile
        int tc[3];
        tile_coords(g, at.tile, tc);
        // lane q: the range of neighbour q where particles came from
        int2 nb = make_int2(0, 0);
        {
            const int tx = tc[0] + lane % 3 - 1, ty = tc[1] + (lane / 3) % 3 - 1, tz = tc[2] + lane / 9 - 1;
            if (lane < 27 && ((from >> lane) & 1) && tx >= 0 && ty >= 0 && tz >= 0 && tx < g.ntile[0] && ty < g.ntile[1] &&
                tz < g.ntile[2])
                nb = rg.range[(tz * g.ntile[1] + ty) * g.ntile[0] + tx];
            if (lane == 13) nb = own;
        }
        int ck[kOwnBatches];   // keys of the own range, then cell | rank << 6, or -1
#pragma unroll
        for (int q = 0; q < kOwnBatches; ++q) ck[q] = q * 64 + lane < own.y ? rg.key[own.x + q * 64 + lane] : -1;
        cnt[lane] = 0;
        wave_sync();
        int found = 0, listed = 0;
        // the next 64 keys in slot order: cell | rank << 6 of those of this tile
        auto count = [&](int key) {
            const bool mine = (key >> 6) == at.tile;
            const unsigned long long m = __ballot(mine);
            if (!m) return -1;
            const int c = key & 63;
            unsigned long long same = m;
#pragma unroll
            for (int b = 0; b < 6; ++b) {
                const unsigned long long bits = __ballot((c >> b) & 1);
                same &= ((c >> b) & 1) ? bits : ~bits;
            }
            found += __popcll(m);
            const int rk = __popcll(same & below), base = cnt[c];
            wave_sync();   // all lanes of a cell have read its count before its first one adds to it
            if (mine && rk == 0) cnt[c] = base + __popcll(same);
            wave_sync();
            return mine ? c | (base + rk) << 6 : -1;
        };
        // particles that go to a list in the tile's range of tmp, tmpk
        auto put = [&](int slot, int r) {
            const unsigned long long m = __ballot(r >= 0);
            const int at_list = listed + __popcll(m & below);
            if (r >= 0 && at_list < at.cnt) {
                tmp[at.off + at_list] = slot;
                tmpk[at.off + at_list] = r;
            }
            listed += __popcll(m);
        };
        auto list = [&](int first, int num) {
            for (int u0 = 0; u0 < num; u0 += 64 * 4) {
                int k[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) k[q] = u0 + q * 64 + lane < num ? rg.key[first + u0 + q * 64 + lane] : -1;
#pragma unroll
                for (int q = 0; q < 4; ++q) put(first + u0 + q * 64 + lane, count(k[q]));
            }
        };
        // the far ones wait in the end of that range, which the list reaches
        // only after it has taken as many of them
        const int n_far = from & kFarBit ? far_sorted(Far{rg.moved, g.ntiles}, rg.N, at, tmp, perm + at.off) : 0;
        int far_at = 0;
        auto far_before = [&](int slot) {
            while (far_at < n_far) {
                const int u = far_at + lane, j = u < n_far ? tmp[at.off + at.cnt - n_far + u] : 0x7fffffff;
                const int num = __popcll(__ballot(j < slot));
                put(j, count(j < slot ? rg.key[j] : -1));
                far_at += num;
                if (num < 64) break;
            }
        };
        bool held = own.y <= kOwnBatches * 64;   // the own range's particles stay in ck
        bool all = false;
        // the neighbours' ranges marked and, as 13, the own one
        for (unsigned todo = (from & 0x7ffffffu) | 1u << 13;; todo = 1) {
            for (; todo; todo &= todo - 1) {
                const int q = __ffs((int)todo) - 1;
                const int first = __shfl(nb.x, q), num = __shfl(nb.y, q);
                if (n_far > far_at) far_before(first);
                if (q == 13 && held) {
#pragma unroll
                    for (int i = 0; i < kOwnBatches; ++i) ck[i] = count(ck[i]);
                } else {
                    list(first, num);
                }
            }
            if (n_far > far_at) far_before(0x7fffffff);
            if (found == at.cnt || all) break;
            // a crowded tile whose chain was not taken: all keys
            all = true;
            cnt[lane] = 0;
            wave_sync();
            found = listed = 0;
            held = false;
            nb = make_int2(0, (int)rg.N);
        }
        if (lane == 0) {
            rg.moved[at.tile] = 0;
            rg.count[at.tile] = 0;
        }
        // rank table, then every particle's place
        const int v = cnt[lane];
        cell_cnt[e * 64 + lane] = v;
        int run = 0;
        for (int q = 0; q < 64; ++q) {
            const unsigned long long m = __ballot(v > q);
            if (!m) break;
            if (lane == 0) {
                s_rmask[w][q] = m;
                s_roff[w][q] = run;
            }
            run += __popcll(m);
        }
        wave_sync();
        int* out = perm + at.off;
        if (held) {
#pragma unroll
            for (int q = 0; q < kOwnBatches; ++q)
                if (ck[q] >= 0) out[rank_major_pos(ck[q] & 63, ck[q] >> 6, s_rmask[w], s_roff[w], cnt)] = own.x + q * 64 + lane;
        }
        __threadfence_block();   // the list was written by this wave
        for (int u = lane; u < listed; u += 64) {
            const int r = ((const volatile int*)tmpk)[at.off + u];
            out[rank_major_pos(r & 63, r >> 6, s_rmask[w], s_roff[w], cnt)] = ((const volatile int*)tmp)[at.off + u];
        }
        wave_sync();
    }
}

// The same from the bucketed entries of each tile, which come in no order: by
// placement into the cells and counting, in LDS.
template <int Unused = 0>
__global__ __launch_bounds__(kSortBlock) void k_sort(Far far, int* __restrict__ meta, int* __restrict__ n_halo,
                                                     const ActiveTile* __restrict__ active, int* __restrict__ tmp, const int* __restrict__ tmpk,
                                                     int* __restrict__ perm, int* __restrict__ cell_cnt)
{
    constexpr int NT = kSortBlock, U = (kSortCap + NT - 1) / NT;
    __shared__ TileSort s;
    const int n_active = meta[0];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if (blockIdx.x == 0 && tid == 0) halo_take(n_halo, meta);
    for (int it = 0;; ++it) {
        const int e = tile_entry(it, n_active);
        if (e < 0) break;
        const ActiveTile at = active[e];
        if (tid < 64) {
            s.cnt[tid] = 0;
            s.cur[tid] = 0;
        }
        if (tid == 0) {   // what the last step marked is not used here
            far.moved[at.tile] = 0;
            far.head(at.tile) = -1;
        }
        const bool in_lds = at.cnt <= kSortCap;
        // a tile that fits LDS keeps its entries in registers: one batch of loads
        int cc[U], cj[U];
        if (in_lds)
#pragma unroll
            for (int q = 0; q < U; ++q) {
                const int u = q * NT + tid;
                cc[q] = u < at.cnt ? tmpk[at.off + u] & 63 : -1;   // the cell is the low 6 bits of the key
                cj[q] = u < at.cnt ? tmp[at.off + u] : 0;
            }
        __syncthreads();
        if (in_lds) {
#pragma unroll
            for (int q = 0; q < U; ++q)
                if (cc[q] >= 0) atomicAdd(&s.cnt[cc[q]], 1);
        } else {
            for (int k = tid; k < at.cnt; k += NT) atomicAdd(&s.cnt[tmpk[at.off + k] & 63], 1);
        }
        __syncthreads();
        if (w == 0) {
            tile_sort_scan(s, lane);
            cell_cnt[e * 64 + lane] = s.cnt[lane];
        }
        __syncthreads();
        if (in_lds) {
#pragma unroll
            for (int q = 0; q < U; ++q)
                if (cc[q] >= 0) tile_sort_place(s, true, cc[q], cj[q], perm + at.off);
        } else {
            for (int k = tid; k < at.cnt; k += NT) tile_sort_place(s, false, tmpk[at.off + k] & 63, tmp[at.off + k], perm + at.off);
        }
        tile_sort_finish<NT>(s, in_lds, at.cnt, perm + at.off, tmp + at.off);
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// 3-D: P2G
// ---------------------------------------------------------------------------

// P2G of one wave, lane = cell: round r takes the particle of rank r of every
// cell that has one; the lanes of a round read adjacent slots.  A cell's
// particles all hit the same 27 nodes, so a lane sums them in registers: the
// momentum components [A0, A1) (and the mass when MASS; with QV those of the
// momentum without the internal force, node arrays 1 + D + a, for FLIP), then
// adds its sums to the wave's own node arrays, lanes on distinct nodes per
// offset, ordered by wave_sync.  Slots are fetched two rounds ahead and
// particles one.
template <class T, int D, int MAT, int A0, int A1, bool MASS, bool QV, bool NTL>
__device__ __forceinline__ void p2g_wave(const Phys<T>& P, const PView<T>& cur, const int* __restrict__ perm_tile, int mycnt,
                                         const int lb[3], const int gb[3], T (*node)[TileShape<D>::NB])
{
    static_assert(!(MASS && QV), "the mass travels with the momentum including the force");
    constexpr int NK = (D == 3) ? 27 : 9, NB = TileShape<D>::NB;
    constexpr int M = MASS ? 1 : 0;
    constexpr int NQ = M + A1 - A0;                          // node values of this wave
    constexpr int Q0 = M ? 0 : (QV ? 1 + D + A0 : 1 + A0);   // its first node array
    const int lane = threadIdx.x & 63;
    for (int i = lane; i < NQ * NB; i += 64) (&node[Q0][0])[i] = T(0);
    T acc[NK][NQ];
#pragma unroll
    for (int k = 0; k < NK; ++k)
#pragma unroll
        for (int q = 0; q < NQ; ++q) acc[k][q] = T(0);
    // slot of this lane's particle of rank r: the particles of earlier ranks,
    // then those of rank r in earlier cells (called by the lanes that still have
    // particles, in step)
    int before = 0;
    auto slot = [&](int r) {
        const unsigned long long m = __ballot(mycnt > r);
        const int pos = before + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
        before += __popcll(m);
        return mycnt > r ? perm_tile[pos] : 0;
    };
    int j1 = slot(0);
    P2GIn<T, D, MAT, A0, A1, NTL> nx;
    if (mycnt > 0) nx.load(cur, j1);
    j1 = slot(1);
    wave_sync();
    for (int r = 0; r < mycnt; ++r) {
        const P2GIn<T, D, MAT, A0, A1, NTL> in = nx;
        const int j = j1;
        j1 = slot(r + 2);
        if (r + 1 < mycnt) nx.load(cur, j);
        // the products go straight into the sums (one FMA each)
        p2g_particle<T, D, MAT, A0, A1, !QV>(P, in, lb, gb, [&](int k, int, T wx, T mw, T wyz, const T* U, const T* Ex) {
            if constexpr (MASS) acc[k][0] = fma(wx, mw, acc[k][0]);
#pragma unroll
            for (int a = 0; a < A1 - A0; ++a) acc[k][M + a] = fma(wyz, Ex[a], fma(wx, U[a], acc[k][M + a]));
        });
    }
#pragma unroll
    for (int k = 0; k < NK; ++k) {
        int n = block_node<D>(lb, k);
        T cv[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) cv[q] = node[Q0 + q][n];
#pragma unroll
        for (int q = 0; q < NQ; ++q) node[Q0 + q][n] = cv[q] + acc[k][q];
        wave_sync();
    }
}

// One tile per workgroup, whose waves share the tile's particles and split the
// node values, so that the sums fit registers: mass and momentum x | the other
// components; with FLIP the same again for the momentum without the internal
// force.  No wave waits for another: each clears, sums and writes out its own
// node arrays.  NTL: the particles are read with the non-temporal hint.
// What bounds it is reading the particles: cylinder, 2,780,000 particles,
// binary32 94 us with the sort inside -> 72 (234 MB of state it must read, 260
// to 330 MB moved), binary64 190 (one wave, LDS atomics at 4 lanes a clock) ->
// 143, FLIP binary64 (635,000) 90 -> 50.
template <class T, int D, int MAT, bool FL, bool NTL>
__global__ __launch_bounds__((kP2GBlock<FL>)) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 3 : 2))) void k_p2g(Geo g, Phys<T> P, const int* __restrict__ meta,
                                                const ActiveTile* __restrict__ active, const int* __restrict__ cell_cnt,
                                                PView<T> cur, const int* __restrict__ perm,
                                                T* __restrict__ part)
{
    constexpr int TE = TileShape<D>::TE, NB = TileShape<D>::NB;
    constexpr int NV = FL ? 2 * D + 1 : D + 1;          // node values per block node
    __shared__ T s_node[NV][NB];
    const int n_active = meta[0];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int it = 0;; ++it) {
        int e = tile_entry(it, n_active);
        if (e < 0) break;
        const ActiveTile at = active[e];
        const int mycnt = cell_cnt[e * 64 + lane];
        int tc[3];
        tile_coords(g, at.tile, tc);
        // The lane's cell, made opaque to the compiler for this tile: what is
        // derived from it (node offsets, LDS addresses) is then formed per
        // tile instead of being hoisted out of the tile loop, where it would
        // hold registers through the particle loop.
        int cl = lane;
        asm volatile("" : "+v"(cl));
        int lb[3], gb[3];
        lb[0] = cl % TE;
        lb[1] = (cl / TE) % TE;
        lb[2] = (D == 3) ? cl / (TE * TE) : 0;
#pragma unroll
        for (int a = 0; a < 3; ++a) gb[a] = tc[a] * TE + lb[a] - g.G;
        T (*node)[NB] = s_node;
        const int* pt = perm + at.off;
        int q0 = 0, q1 = NV;                            // this wave's node arrays
        if (w == 0) {
            p2g_wave<T, D, MAT, 0, 1, true, false, NTL>(P, cur, pt, mycnt, lb, gb, node);
            q1 = 2;
        } else if (w == 1) {
            p2g_wave<T, D, MAT, 1, D, false, false, NTL>(P, cur, pt, mycnt, lb, gb, node);
            q0 = 2, q1 = 1 + D;
        } else if constexpr (FL) {
            if (w == 2) {
                p2g_wave<T, D, MAT, 0, 1, false, true, NTL>(P, cur, pt, mycnt, lb, gb, node);
                q0 = 1 + D, q1 = 2 + D;
            } else {
                p2g_wave<T, D, MAT, 1, D, false, true, NTL>(P, cur, pt, mycnt, lb, gb, node);
                q0 = 2 + D;
            }
        }
        wave_sync();
        T* dst = part + (long long)e * NV * NB;
        for (int i = q0 * NB + lane; i < q1 * NB; i += 64) dst[i] = (&s_node[0][0])[i];
        wave_sync();
    }
}

// ---------------------------------------------------------------------------
// 2-D: the sort and P2G of a tile in one kernel
//
// A 2-D step is short of work, not of bandwidth: 8,192 particles are 40 tiles
// on 256 CUs, and a step was five launches (scan, bucket, P2G, grid, G2P), each
// a chain of dependent memory round trips of about a microsecond.  Two launches
// remain: this kernel, and G2P, which forms its tile's nodal velocities itself.
//
// Where the previous step's layout is known (GATHER), a tile's particles are
// found without a scan and a scatter over the grid.  The previous G2P left the
// particles of every tile in one range of slots and their new keys beside them,
// and a particle moves at most to a neighbouring tile (a cell is the limit of a
// step, a tile is eight), so a workgroup reads the keys of the nine ranges
// around its tile and picks its own; its offset is the sum of the counts of
// the tiles before it, at most kSmallTiles of them.  The first keys of a range
// are also kept in a row per tile, whose place is known without the range, so
// counts, ranges and keys come in one round trip (G2P likewise finds its
// particles in a row of perm).  A workgroup that finds
// fewer than its tile's count (particles moved further, in a step beyond the
// CFL limit) takes the rest from their chain (see Far).  The order inside the tile is by cell and previous
// slot, whatever order they were found in, so both ways of finding give the
// same permutation and, from there, the same bits.
// ---------------------------------------------------------------------------

// Threads per tile where tiles are many and waves, not latency, are short
// (kSortMany2: binary64, 131,072 particles, 256 threads 37.8 us a step, 128 36.1,
// 64 38.6), and fewer still in binary64 past kNarrow2 particles, here and in G2P
// (kG2PNarrow2): the registers leave two to three waves per SIMD, and those of
// one tile wait for each other.  A step of fluid, sand and sand with FLIP, wide
// and narrow: 122,500 particles 32 and 40, 40 and 52, 43 and 57 us; 494,900 67 and
// 59, 83 and 77, 91 and 84; 3.96 M 366 and 317, 476 and 421, 546 and 472.
constexpr int kSortMany2 = 128;
template <class T> constexpr int kSortNarrow2 = sizeof(T) == 8 ? 64 : kSortMany2;
constexpr long long kNarrow2 = 262144;

// Tile of a workgroup when there is one per tile: a contiguous chunk of tiles
// on each XCD (workgroup b runs on XCD b % 8).  -1 past the end.
__device__ __forceinline__ int tile_of_block(int ntiles)
{
    const int chunk = (ntiles + 7) / 8;
    const int lb = blockIdx.x / 8, t = (blockIdx.x % 8) * chunk + lb;
    return lb < chunk && t < ntiles ? t : -1;
}

// One tile per workgroup of NW waves (four; two where tiles are many).  After
// the sort, wave w takes the particles of rank w, w + NW, ... of every cell,
// lane = cell: a lane sums its
// particles in registers (they all hit the same nine nodes), then adds to its
// wave's own copy of the tile's node block, lanes on distinct nodes per offset;
// the copies are summed in a fixed order.  With four particles per cell a wave
// of four has one round, where one wave (binary64, LDS atomics) had four.
// A step of the 2-D dam-break before the water moves, 8,192 / 32,768 / 73,728
// particles: binary32 24.1 / 25.6 / 28.5 -> 13.8 / 17.6 / 18.6 us, binary64 28.8 /
// 31.0 / 35.1 -> 15.1 / 20.2 / 22.6; over 1000 steps of 8,192 26.2 -> 16.7 and 32.1 ->
// 17.8.  This kernel takes 7.7 us of it at 8,192 particles and
// G2P 6.2; what bounds both is the chain of launch, two memory round trips,
// LDS phases and the drain of the stores.
template <class T, int MAT, bool FL, bool GATHER, int NT>
__global__ __launch_bounds__(NT) void k_sort_p2g2(Geo g, Phys<T> P, Ranges rg, int* __restrict__ meta,
                                                           ActiveTile* __restrict__ active, int* __restrict__ tile_slot,
                                                           int* __restrict__ tmp, int* __restrict__ tmpk, PView<T> cur,
                                                           int* __restrict__ perm, T* __restrict__ part)
{
    constexpr int D = 2, TE = TileShape<D>::TE, NB = TileShape<D>::NB, NW = NT / 64;
    constexpr int NV = FL ? 2 * D + 1 : D + 1;   // node values per block node
    constexpr int NK = 9;
    __shared__ T s_node[NW][NV][NB];
    __shared__ TileSort ts;
    __shared__ int s_sum[2][NW], s_first[9], s_num[9], s_far;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int n_active = GATHER ? 0 : meta[0];
    constexpr int U = GATHER ? 9 : (kSortCap + NT - 1) / NT;
    static_assert(!GATHER || kTileRow == NT, "a thread holds one entry of each tile's row");
    for (int it = 0;; ++it) {
        ActiveTile at;
        int cj[U], cc[U];   // candidates: slot, and key, then cell or -1
        if (tid < 64) {
            ts.cnt[tid] = 0;
            ts.cur[tid] = 0;
        }
        if constexpr (GATHER) {
            const int t = it == 0 ? tile_of_block(g.ntiles) : -1;
            if (t < 0) break;
            const int own = rg.count[t];
            const int ty = t / g.ntile[0], tx = t - ty * g.ntile[0];
            // the row of a neighbour outside the grid is read as the tile's own and not used
#pragma unroll
            for (int q = 0; q < U; ++q) {
                const int nx = tx + q % 3 - 1, ny = ty + q / 3 - 1;
                const bool in = nx >= 0 && ny >= 0 && nx < g.ntile[0] && ny < g.ntile[1];
                cc[q] = rg.tile_key[(in ? ny * g.ntile[0] + nx : t) * kTileRow + tid];
            }
            if (tid < 9) {
                const int nx = tx + tid % 3 - 1, ny = ty + tid / 3 - 1;
                const bool in = nx >= 0 && ny >= 0 && nx < g.ntile[0] && ny < g.ntile[1];
                const int2 r = in ? rg.range[ny * g.ntile[0] + nx] : make_int2(0, 0);
                s_first[tid] = r.x;
                s_num[tid] = r.y;
            }
            int s = 0, a = 0;
            for (int i = tid; i < t; i += NT) {
                const int c = rg.count[i];
                s += c;
                a += c > 0;
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                s += __shfl_xor(s, o);
                a += __shfl_xor(a, o);
            }
            if (lane == 0) {
                s_sum[0][w] = s;
                s_sum[1][w] = a;
            }
            __syncthreads();
            s = a = 0;
#pragma unroll
            for (int i = 0; i < NW; ++i) {
                s += s_sum[0][i];
                a += s_sum[1][i];
            }
            at.tile = t;
            at.off = s;
            at.cnt = own;
            at.pad = 0;
            if (tid == 0) {
                tile_slot[t] = own > 0 ? a : -1;
                if (own > 0) active[a] = at;
                rg.range_next[t] = make_int2(s, own);
                rg.count_next[t] = 0;
                if (t == g.ntiles - 1) {
                    meta[0] = a + (own > 0);
                    meta[1] = s + own;
                }
            }
            if (own == 0) break;
        } else {
            const int e = tile_entry(it, n_active);
            if (e < 0) break;
            at = active[e];
            if (rg.moved && tid == 0) Far{rg.moved, g.ntiles}.head(at.tile) = -1;   // not used here
            __syncthreads();
        }
        const bool in_lds = at.cnt <= kSortCap;
        // Candidates: the keys of the nine ranges (or all keys), or the tile's
        // bucketed entries.  A batch is U per thread, loaded together (of each
        // range kTileRow); where one batch holds them all it stays in registers
        // from the histogram to the placement.
        bool all = false;
        auto batch = [&](int u0) {
            if constexpr (GATHER) {
#pragma unroll
                for (int q = 0; q < U; ++q) {
                    const int u = all ? u0 * U + q * NT + tid : u0 + tid;
                    cj[q] = all ? (u < (int)rg.N ? u : -1) : (u < s_num[q] ? s_first[q] + u : -1);
                }
                if (u0 > 0 || all)
#pragma unroll
                    for (int q = 0; q < U; ++q) cc[q] = cj[q] >= 0 ? rg.key[cj[q]] : -1;
#pragma unroll
                for (int q = 0; q < U; ++q) cc[q] = cj[q] >= 0 && (cc[q] >> 6) == at.tile ? cc[q] & 63 : -1;
            } else {
#pragma unroll
                for (int q = 0; q < U; ++q) {
                    const int u = u0 * U + q * NT + tid;
                    cc[q] = u < at.cnt ? tmpk[at.off + u] & 63 : -1;
                    cj[q] = u < at.cnt ? tmp[at.off + u] : -1;
                }
            }
        };
        // entries to go through, in units of U
        int total = (at.cnt + U - 1) / U;
        if constexpr (GATHER) {
            total = 0;
#pragma unroll
            for (int b = 0; b < 9; ++b) total = max(total, s_num[b]);
        }
        int n_far = 0;   // particles of the tile's chain, listed in its range of tmp
        for (;;) {
            for (int u0 = 0; u0 < total; u0 += NT) {
                batch(u0);
#pragma unroll
                for (int q = 0; q < U; ++q)
                    if (cc[q] >= 0) atomicAdd(&ts.cnt[cc[q]], 1);
            }
            __syncthreads();
            if (w == 0) tile_sort_scan(ts, lane);
            __syncthreads();
            if (!GATHER || all || ts.found == at.cnt) break;
            __syncthreads();   // all waves have read ts.found, which the first forms anew
            if (w == 0) {
                // some came from further away: along their chain, one by one
                const Far far{rg.moved, g.ntiles};
                int j = __builtin_amdgcn_readfirstlane(far.head(at.tile)), n = 0;
                if (far_scans_all(at.cnt, rg.N)) j = -1;
                for (; j >= 0 && n < at.cnt; ++n) {
                    if (lane == 0) {
                        tmp[at.off + n] = j;
                        atomicAdd(&ts.cnt[rg.key[j] & 63], 1);
                    }
                    j = __builtin_amdgcn_readfirstlane(far.next(j));
                }
                if (lane == 0) {
                    far.head(at.tile) = -1;
                    s_far = n;
                }
                wave_sync();
                tile_sort_scan(ts, lane);
            }
            __syncthreads();
            n_far = s_far;
            if (ts.found == at.cnt) break;
            // a crowded tile whose chain was not taken
            __syncthreads();
            if (tid < 64) ts.cnt[tid] = 0;
            n_far = 0;
            all = true;
            total = (int)((rg.N + U - 1) / U);
            __syncthreads();
        }
        // cell-major placement, then the rank inside the cell by previous slot
        for (int u0 = 0; u0 < total; u0 += NT) {
            if (total > NT) {
                if (GATHER && u0 == 0 && !all)
#pragma unroll
                    for (int q = 0; q < U; ++q) cc[q] = u0 + tid < s_num[q] ? rg.key[s_first[q] + tid] : -1;
                batch(u0);
            }
#pragma unroll
            for (int q = 0; q < U; ++q)
                if (cc[q] >= 0) tile_sort_place(ts, in_lds, cc[q], cj[q], perm + at.off);
        }
        if constexpr (GATHER)
            for (int u = tid; u < n_far; u += NT) {
                const int j = tmp[at.off + u];
                tile_sort_place(ts, in_lds, rg.key[j] & 63, j, perm + at.off);
            }
        tile_sort_finish<NT>(ts, in_lds, at.cnt, perm + at.off, tmp + at.off);
        const int* sorted = in_lds ? ts.sorted : (perm + at.off);
        if (NT == kTileRow && rg.tile_perm && tid < at.cnt) rg.tile_perm[at.tile * kTileRow + tid] = sorted[tid];
        int tc[3];
        tile_coords(g, at.tile, tc);
        // opaque to the compiler for this tile, so that what is derived from the
        // cell is not hoisted out of the tile loop into registers
        int cl = lane;
        asm volatile("" : "+v"(cl));
        const int lb[3] = {cl % TE, cl / TE, 0};
        const int gb[3] = {tc[0] * TE + lb[0] - g.G, tc[1] * TE + lb[1] - g.G, 0};
        const int mycnt = ts.cnt[cl];
        T acc[NK][NV];
#pragma unroll
        for (int k = 0; k < NK; ++k)
#pragma unroll
            for (int q = 0; q < NV; ++q) acc[k][q] = T(0);
        P2GIn<T, D, MAT> nx;
        if (w < mycnt) nx.load(cur, sorted[rank_major_pos(cl, w, ts.rmask, ts.roff, ts.cnt)]);
        T(*node)[NB] = s_node[w];
        for (int i = lane; i < NV * NB; i += 64) (&node[0][0])[i] = T(0);
        for (int r = w; r < mycnt; r += NW) {
            const P2GIn<T, D, MAT> in = nx;
            if (r + NW < mycnt) nx.load(cur, sorted[rank_major_pos(cl, r + NW, ts.rmask, ts.roff, ts.cnt)]);
            p2g_particle<T, D, MAT, 0, D, true>(P, in, lb, gb, [&](int k, int, T wx, T mw, T wyz, const T* U, const T* Ex) {
                acc[k][0] = fma(wx, mw, acc[k][0]);
#pragma unroll
                for (int a = 0; a < D; ++a) acc[k][1 + a] = fma(wyz, Ex[a], fma(wx, U[a], acc[k][1 + a]));
            });
            if constexpr (FL)
                p2g_particle<T, D, MAT, 0, D, false>(P, in, lb, gb, [&](int k, int, T wx, T, T wyz, const T* U, const T* Ex) {
#pragma unroll
                    for (int a = 0; a < D; ++a) acc[k][1 + D + a] = fma(wyz, Ex[a], fma(wx, U[a], acc[k][1 + D + a]));
                });
        }
        wave_sync();
#pragma unroll
        for (int k = 0; k < NK; ++k) {
            const int n = block_node<D>(lb, k);
            T cv[NV];
#pragma unroll
            for (int q = 0; q < NV; ++q) cv[q] = node[q][n];
#pragma unroll
            for (int q = 0; q < NV; ++q) node[q][n] = cv[q] + acc[k][q];
            wave_sync();
        }
        __syncthreads();
        T* dst = part + (long long)at.tile * NV * NB;
        for (int i = tid; i < NV * NB; i += NT) {
            T s = (&s_node[0][0][0])[i];
#pragma unroll
            for (int k = 1; k < NW; ++k) s += (&s_node[k][0][0])[i];
            dst[i] = s;
        }
        if constexpr (GATHER) break;
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Grid update over the node blocks of the active tiles.  A node shared by
// several blocks is handled by exactly one of them: the first active tile
// among its candidates, own tile first.  Its mass and momentum are the sum of
// the partial blocks that cover it, in that same fixed order.
// ---------------------------------------------------------------------------

// Whether a node's eight candidate blocks are loaded in one batch or two (past
// 16 bytes per block two, the registers would cost waves: binary64 18.8 and
// 18.5 us on the cylinder, FLIP 13.2 and 12.7 on the column).
template <class T, int NS> constexpr int kNodeUnroll = NS * sizeof(T) <= 16 ? 2 : 1;

// Sums the partial blocks over the 64 nodes of an active or a halo tile, one per
// lane: NS of a block's NV values per node.  A node's blocks are those of the
// tile it lies in and of that tile minus one along axes where it is one of the
// first two nodes; the sum takes them in the order of the bits (x first).  With
// one wave per tile every lane has its node; when each active tile went over the
// 216 nodes of its block and left those that another tile owned, 70 % of the
// threads were idle, and a second pass for the nodes past an active tile alone
// took longer than the first (three trips to memory in a row).  The 27 tiles
// around are looked up once, one per lane.  Latency bounds it: the lists, the
// neighbours, the blocks, the stores.  Grid update, block by block and so: 2.78 M
// particles binary32 20.9 -> 15.1 us, binary64 26.0 -> 19.2, 1.92 M 20.6 -> 12.7,
// FLIP binary64 (635,000) 17.2 -> 13.3; its reverse, 1.84 M binary32 26.2 ->
// 15.5, 442,368 binary64 15.7 -> 10.7.
// pre(node) loads what else the node needs; post(I, node, in, sum) writes it.
template <class T, int NV, int NS, class Pre, class Post>
__device__ __forceinline__ void tile_nodes(const Geo& g, int tile, const int* __restrict__ tile_slot,
                                           const T* __restrict__ part, int* around_of, Pre pre, Post post)
{
    constexpr int TE = TileShape<3>::TE, BE = TileShape<3>::BE, NB = TileShape<3>::NB;
    const int lane = threadIdx.x & 63;
    int tc[3];
    tile_coords(g, tile, tc);
    const int around = around_slot(g, tile, tile_slot);
    // the node at l of the block, h tiles up; slot(b): the block of the tile b
    // below the one it lies in (-1: none)
    auto add = [&](const int l[3], const int h[3], auto slot) {
        const int I[3] = {tc[0] * TE + l[0], tc[1] * TE + l[1], tc[2] * TE + l[2]};
        const long long node = node_index(g, I[0], I[1], I[2]);
        const auto in = pre(node);
        bool any = false;
        T sum[NS];
#pragma unroll
        for (int q = 0; q < NS; ++q) sum[q] = T(0);
#pragma unroll kNodeUnroll<T, NS>
        for (int b2 = 0; b2 < 2; ++b2) {
            T v[4][NS];
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int b[3] = {m & 1, m >> 1, b2}, s = slot(b);
                any |= s >= 0;
                const int o[3] = {l[0] + TE * (b[0] - h[0]), l[1] + TE * (b[1] - h[1]), l[2] + TE * (b[2] - h[2])};
                const T* src = part + (long long)s * NV * NB + (o[2] * BE + o[1]) * BE + o[0];
#pragma unroll
                for (int q = 0; q < NS; ++q) v[m][q] = s >= 0 ? src[q * NB] : T(0);
            }
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int q = 0; q < NS; ++q) sum[q] += v[m][q];
        }
        if (any) post(I, node, in, sum);
    };
    {
        const int l[3] = {lane % TE, (lane / TE) % TE, lane / (TE * TE)}, h[3] = {0, 0, 0};
        add(l, h, [&](const int b[3]) {
            const int s = __builtin_amdgcn_readlane(around, 13 - b[0] - 3 * b[1] - 9 * b[2]);
            return (!b[0] || l[0] < 2) && (!b[1] || l[1] < 2) && (!b[2] || l[2] < 2) ? s : -1;
        });
    }
    // Past the last tiles of the grid lie two more layers of nodes, which only a
    // particle beyond the walls reaches.  Each belongs to the first active one of
    // the tiles whose blocks cover it, in the same order.
    const unsigned act = (unsigned)__ballot(around >= 0);
    if (!((act >> 13) & 1) || (tc[0] + 1 < g.ntile[0] && tc[1] + 1 < g.ntile[1] && tc[2] + 1 < g.ntile[2])) return;
    if (lane < 27) around_of[lane] = around;
    wave_sync();
    for (int j0 = 0; j0 < NB - 64; j0 += 64) {
        // the block's nodes past the tile along z (72), else y (48), else x (32)
        const int j = j0 + lane;
        int l[3];
        if (j < 72) l[0] = j % 6, l[1] = (j / 6) % 6, l[2] = 4 + j / 36;
        else if (j < 120) l[0] = (j - 72) % 6, l[1] = 4 + ((j - 72) / 6) % 2, l[2] = (j - 72) / 12;
        else l[0] = 4 + (j - 120) % 2, l[1] = ((j - 120) / 2) % 4, l[2] = (j - 120) / 8;
        const int h[3] = {l[0] >= TE, l[1] >= TE, l[2] >= TE};
        auto place = [&](const int b[3]) {
            const bool covers = (!b[0] || l[0] - TE * h[0] < 2) && (!b[1] || l[1] - TE * h[1] < 2) &&
                                (!b[2] || l[2] - TE * h[2] < 2);
            return covers ? 13 + h[0] - b[0] + 3 * (h[1] - b[1]) + 9 * (h[2] - b[2]) : 31;   // bit 31 of act is clear
        };
        int owner = -1;
#pragma unroll
        for (int msk = 7; msk >= 0; --msk) {
            const int b[3] = {msk & 1, (msk >> 1) & 1, msk >> 2};
            if ((act >> place(b)) & 1) owner = msk;
        }
        const bool past = (h[0] && tc[0] + 1 == g.ntile[0]) || (h[1] && tc[1] + 1 == g.ntile[1]) ||
                          (h[2] && tc[2] + 1 == g.ntile[2]);
        const bool mine = j < NB - 64 && past && owner == (h[0] | h[1] << 1 | h[2] << 2);
        if (mine)
            add(l, h, [&](const int b[3]) {
                const int q = place(b);
                return (act >> q) & 1 ? around_of[q] : -1;
            });
    }
    wave_sync();
}

// Velocity of a node of mass m > 0 and momentum p after the grid update, the
// walls and the resting obstacles (Sec. 4.2.1); vt: before the walls.
template <class T, int D>
__device__ __forceinline__ void node_velocity(const Geo& g, const Phys<T>& P, const int I[3], T m, const T p[D], T v[D],
                                              T vt[D])
{
#pragma unroll
    for (int a = 0; a < D; ++a) vt[a] = v[a] = p[a] / m + P.dt * P.g[a];
#pragma unroll
    for (int a = 0; a < D; ++a) {
        int ip = I[a] - g.G;
        if (ip <= 0) {
            T mu = P.wall_mu[2 * a];
            if (a == D - 1 && P.floor_mu) {
                int fx = min(I[0], g.box[0] - 1);
                int fi = (D == 3) ? min(I[1], g.box[1] - 1) * P.floor_stride + fx : fx;
                mu = P.floor_mu[fi];
            }
            wall_node<T, D>(P.wall_mode[2 * a], mu, a, T(-1), v);
        }
        if (ip >= g.n[a]) wall_node<T, D>(P.wall_mode[2 * a + 1], P.wall_mu[2 * a + 1], a, T(1), v);
    }
    if (P.n_obst > 0) {
        double xi[D];
#pragma unroll
        for (int a = 0; a < D; ++a) xi[a] = double(I[a] - g.G) * P.obst_h;
        obstacle_node<T, D>(P, xi, v);
    }
}

// With FL (FLIP) the partial blocks also hold the momentum without the
// internal force, and gvo receives the velocity before the update,
// v_i^n = that / m_i (0 where m_i = 0).
template <class T, int D, bool FL>
__global__ __launch_bounds__(kGridBlock) void k_grid(Geo g, Phys<T> P, const int* __restrict__ meta,
                                                 const ActiveTile* __restrict__ active,
                                                 const int* __restrict__ tile_slot, const T* __restrict__ part,
                                                 T* __restrict__ gv, T* __restrict__ gmass, T* __restrict__ gvt,
                                                 T* __restrict__ gvo)
{
    constexpr int NV = FL ? 2 * D + 1 : D + 1;
    __shared__ int s_around[kGridBlock / 64][27];
    for (int it = 0;; ++it) {
        const int tile = node_tile<kGridBlock / 64>(it, meta, active, g.ntiles);
        if (tile < 0) break;
        tile_nodes<T, NV, NV>(
            g, tile, tile_slot, part, s_around[threadIdx.x >> 6], [](long long) { return 0; },
            [&](const int I[3], long long node, int, const T sum[NV]) {
                const T m = sum[0];
                T v[D], vt[D];
#pragma unroll
                for (int a = 0; a < D; ++a) v[a] = vt[a] = T(0);
                if (m > T(0)) node_velocity<T, D>(g, P, I, m, sum + 1, v, vt);
                if (gvt)
#pragma unroll
                    for (int a = 0; a < D; ++a) gvt[a * g.NN + node] = vt[a];
#pragma unroll
                for (int a = 0; a < D; ++a) gv[a * g.NN + node] = v[a];
                if constexpr (FL)
#pragma unroll
                    for (int a = 0; a < D; ++a) gvo[a * g.NN + node] = m > T(0) ? sum[1 + D + a] / m : T(0);
                if (P.keep_grid) gmass[node] = m;
            });
    }
}

// ---------------------------------------------------------------------------
// Gathers over the stencil
// ---------------------------------------------------------------------------

// The per-axis factors of a particle's weights: w, w dd (dd = x_i - x_p) and
// d phi / dx.
template <class T, int D>
struct AxisFactors {
    T w[D][3], wd[D][3], dw[D][3];
    __device__ __forceinline__ void set(int a, T f, T inv, T h)
    {
        weights_from_f(f, inv, w[a], dw[a]);
#pragma unroll
        for (int k = 0; k < 3; ++k) wd[a][k] = w[a][k] * ((T(k) - f) * h);
    }
};

// Sums of a node field over the stencil with the weights of all axes but one:
// R[b][k] = sum over the nodes with offset k along b of field * (product of the
// other axes' w).  Every gather of the field is a sum over k of these with one
// axis's own factors: sum phi field = sum_k w_0 R_0, sum phi field dd_b =
// sum_k wd_b R_b, sum field d_b phi = sum_k dw_b R_b; 81 multiply-adds for the
// R and 21 for the seven sums of a component, where summing each of the seven
// line by line was 144 and the lines' factors.  The barrier after each plane
// keeps the compiler from hoisting all LDS reads of the stencil (registers,
// occupancy).
template <class B, class T, int D>
__device__ __forceinline__ void axis_sums(const T (&f)[B::LN], int n0, const AxisFactors<T, D>& A, T R[D][3])
{
    constexpr int LY = B::LY, LZ = B::LZ;
    if constexpr (D == 2) {
#pragma unroll
        for (int k = 0; k < 3; ++k) R[0][k] = R[1][k] = T(0);
#pragma unroll
        for (int ky = 0; ky < 3; ++ky)
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) {
                const T p = f[n0 + ky * LY + kx];
                R[0][kx] = fma(A.w[1][ky], p, R[0][kx]);
                R[1][ky] = fma(A.w[0][kx], p, R[1][ky]);
            }
    } else {
        T xy[3][3];   // summed along z
#pragma unroll
        for (int ky = 0; ky < 3; ++ky)
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) xy[ky][kx] = T(0);
#pragma unroll
        for (int kz = 0; kz < 3; ++kz) {
            R[2][kz] = T(0);
#pragma unroll
            for (int ky = 0; ky < 3; ++ky) {
                T x = T(0);   // summed along x
#pragma unroll
                for (int kx = 0; kx < 3; ++kx) {
                    const T p = f[n0 + kz * LZ + ky * LY + kx];
                    x = fma(A.w[0][kx], p, x);
                    xy[ky][kx] = fma(A.w[2][kz], p, xy[ky][kx]);
                }
                R[2][kz] = fma(A.w[1][ky], x, R[2][kz]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) R[0][k] = R[1][k] = T(0);
#pragma unroll
        for (int ky = 0; ky < 3; ++ky)
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) {
                R[0][kx] = fma(A.w[1][ky], xy[ky][kx], R[0][kx]);
                R[1][ky] = fma(A.w[0][kx], xy[ky][kx], R[1][ky]);
            }
    }
}

template <class T>
__device__ __forceinline__ T dot3(const T a[3], const T b[3])
{
    return fma(a[2], b[2], fma(a[1], b[1], a[0] * b[0]));
}

// ---------------------------------------------------------------------------
// G2P + kinematics + constitutive
// ---------------------------------------------------------------------------

// Nodal velocities of a tile's LDS block (the tile's nodes and its halo), NPT
// block nodes per thread: thread t takes nodes t, t + NT, ...
template <class T, int D, int NPT, int NT>
__device__ __forceinline__ void g2p_block_load(const Geo& g, const T* __restrict__ gv, int tile, int tid,
                                               T r[D][NPT])
{
    constexpr int TE = TileShape<D>::TE, BE = TileShape<D>::BE, NB = TileShape<D>::NB;
    int tc[3];
    tile_coords(g, tile, tc);
#pragma unroll
    for (int p = 0; p < NPT; ++p) {
        const int i = tid + p * NT;
        if (i < NB) {
            int l0 = i % BE, l1 = (i / BE) % BE, l2 = (D == 3) ? i / (BE * BE) : 0;
            long long node = node_index(g, tc[0] * TE + l0, tc[1] * TE + l1, (D == 3) ? tc[2] * TE + l2 : 0);
#pragma unroll
            for (int a = 0; a < D; ++a) r[a][p] = gv[a * g.NN + node];
        }
    }
}

// 2-D: what G2P needs to form its tile's nodal velocities from P2G's partial
// blocks, and where they are kept.
template <class T>
struct Nodes2 {
    const T* part;          // partial block of each tile (indexed by tile)
    const int* tile_slot;
    const int2* range;      // one workgroup per tile: each tile's particles,
    const int* tile_perm;   // the first kTileRow entries of its perm
    int* tile_key;          // and of the new keys
    T *gv, *gmass, *gvt, *gvo;
};

// Sum of NV values over the partial blocks (one per tile, stride NS values per
// node) that cover node `tid` of a tile's block, own tile first, then the tile
// below along x, y and both.  I: the node; returns its owner, the first active
// tile that covers it.  Blocks are loaded before it is known which tiles are
// active: one round trip.
template <class T, int NV, int NS>
__device__ __forceinline__ int block_sum2(const Geo& g, const int* __restrict__ tile_slot, const T* __restrict__ part, int tile,
                                          int tid, int I[3], T sum[NV])
{
    constexpr int D = 2, TE = TileShape<D>::TE, BE = TileShape<D>::BE, NB = TileShape<D>::NB, NC = 4;
    int tc[3];
    tile_coords(g, tile, tc);
    const int l[2] = {tid % BE, tid / BE};
    int own[2];
    bool down[2];
    I[2] = 0;
#pragma unroll
    for (int a = 0; a < D; ++a) {
        I[a] = tc[a] * TE + l[a];
        own[a] = I[a] / TE;
        down[a] = (I[a] % TE < 2) && own[a] >= 1;
    }
    int tl[NC], slot[NC];
    T val[NC][NV];
#pragma unroll
    for (int msk = 0; msk < NC; ++msk) {
        const int cx = own[0] - (msk & 1), cy = own[1] - (msk >> 1);
        const bool ok = (!(msk & 1) || down[0]) && (!(msk >> 1) || down[1]) && cx < g.ntile[0] && cy < g.ntile[1];
        tl[msk] = ok ? cy * g.ntile[0] + cx : -1;
        const int src = ok ? tl[msk] : tile;
        const int li = ok ? (I[1] - cy * TE) * BE + I[0] - cx * TE : 0;
        slot[msk] = tile_slot[src];
        const T* p = part + (long long)src * NS * NB + li;
#pragma unroll
        for (int q = 0; q < NV; ++q) val[msk][q] = p[q * NB];
    }
    int des = -1;
#pragma unroll
    for (int q = 0; q < NV; ++q) sum[q] = T(0);
#pragma unroll
    for (int msk = 0; msk < NC; ++msk)
        if (tl[msk] >= 0 && slot[msk] >= 0) {
            if (des < 0) des = tl[msk];
#pragma unroll
            for (int q = 0; q < NV; ++q) sum[q] += val[msk][q];
        }
    return des;
}

// The node update of k_grid for the 100 nodes of one tile's block, one per
// thread, into LDS.  A node shared by several tiles is formed by each of them
// from the same sums in the same order (1.56 updates per node); its owner
// stores it.
template <class T, bool FL>
__device__ __forceinline__ void node_block2(const Geo& g, const Phys<T>& P, const Nodes2<T>& nd, int tile, int tid,
                                            T (&s_v)[2][TileShape<2>::NB], T (*s_vo)[FL ? TileShape<2>::NB : 1])
{
    constexpr int D = 2, NB = TileShape<D>::NB, NV = FL ? 2 * D + 1 : D + 1;
    if (tid >= NB) return;
    int I[3];
    T sum[NV];
    const int des = block_sum2<T, NV, NV>(g, nd.tile_slot, nd.part, tile, tid, I, sum);
    const T m = sum[0];
    T v[D] = {T(0), T(0)}, vt[D] = {T(0), T(0)};
    if (m > T(0)) node_velocity<T, D>(g, P, I, m, &sum[1], v, vt);
    const long long node = node_index(g, I[0], I[1], 0);
    const bool keep = des == tile;
#pragma unroll
    for (int a = 0; a < D; ++a) {
        s_v[a][tid] = v[a];
        if (keep) {
            nd.gv[a * g.NN + node] = v[a];
            if (nd.gvt) nd.gvt[a * g.NN + node] = vt[a];
        }
        if constexpr (FL) {
            const T vo = m > T(0) ? sum[1 + D + a] / m : T(0);
            s_vo[a][tid] = vo;
            if (keep && nd.gvo) nd.gvo[a * g.NN + node] = vo;
        }
    }
    if (keep && P.keep_grid) nd.gmass[node] = m;
}

// The transfer (App. B) sets the new velocity and the carried matrix C:
// APIC C = (4/h^2) sum phi v_i (x_i - x_p)^T, TPIC C = the velocity gradient,
// PIC and FLIP C = 0; FLIP (FL) also gathers the grid velocity before the
// update, gvo, and blends: v' = sum phi v_i + alpha (v_p - sum phi v_i^n).
// BYTILE (2-D grids of few tiles): one workgroup per tile, else over the active
// list.
template <class T, int D, int MAT, int XF, bool BYTILE, int NT = kG2PBlock<T, D>>
__global__ __launch_bounds__(NT) void k_g2p(Geo g, Phys<T> P, const int* __restrict__ meta,
                                                const ActiveTile* __restrict__ active, const int* __restrict__ perm,
                                                PView<T> cur, PView<T> nxt, const T* __restrict__ gv,
                                                const T* __restrict__ gvo,
                                                int* __restrict__ key_out, int* __restrict__ count,
                                                int* __restrict__ status, const T* __restrict__ eps_in,
                                                T* __restrict__ eps_out, Nodes2<T> nd, int* __restrict__ moved)
{
    constexpr int TE = TileShape<D>::TE, BE = TileShape<D>::BE, NB = TileShape<D>::NB;
    constexpr int NS = D * (D + 1) / 2;
    constexpr int NPT = (NB + NT - 1) / NT;   // block nodes per thread
    constexpr bool FL = XF == XF_FLIP;
    __shared__ T s_v[D][NB];
    __shared__ T s_vo[FL ? D : 1][FL ? NB : 1];
    static_assert(!BYTILE || (D == 2 && NT == kTileRow), "a thread holds one entry of its tile's row");
    const int n_active = BYTILE ? 0 : meta[0];
    const int tid = threadIdx.x;
    const long long cap = cur.cap;
    // With kG2PPrefetch, the next tile's node velocities are loaded into
    // registers while this tile's particles are processed (and its
    // active-list entry one tile earlier still); otherwise each tile loads its
    // own block at its top.
    constexpr bool PF = kG2PPrefetch<T> && !FL && D == 3;
    int e = __builtin_amdgcn_readfirstlane(BYTILE ? tile_of_block(g.ntiles) : tile_entry(0, n_active));
    if (e < 0) return;
    ActiveTile at;
    int j_row = 0;
    if constexpr (BYTILE) {
        const int2 r = nd.range[e];
        j_row = nd.tile_perm[e * kTileRow + tid];
        at.tile = e;
        at.off = r.x;
        at.cnt = r.y;
        if (at.cnt == 0) return;
    } else {
        at = active[e];
    }
    T pre[D][NPT];
    if (PF) g2p_block_load<T, D, NPT, NT>(g, gv, at.tile, tid, pre);
    int en = BYTILE ? -1 : __builtin_amdgcn_readfirstlane(tile_entry(1, n_active));
    int next_tile = (PF && en >= 0) ? active[en].tile : 0;
    for (int it = 0; e >= 0; ++it) {
        // 2-D: a thread's first particle is on its way while the nodes are formed
        constexpr int NG = mat_has_F(MAT) ? D * D : 1;
        int j_first = 0, pid_first = 0;
        T x_first[D], g_first[NG];
        if constexpr (D == 2) {
            if (tid < at.cnt) {
                j_first = BYTILE ? j_row : ld_once(&perm[at.off + tid]);
#pragma unroll
                for (int a = 0; a < D; ++a) x_first[a] = ld_once(&cur.x[a * cap + j_first]);
#pragma unroll
                for (int q = 0; q < NG; ++q) g_first[q] = ld_once(&cur.G[q * cap + j_first]);
                pid_first = ld_once(&cur.pid[j_first]);
            }
            node_block2<T, FL>(g, P, nd, at.tile, tid, s_v, s_vo);
        }
        if (!PF && D == 3) g2p_block_load<T, D, NPT, NT>(g, gv, at.tile, tid, pre);
        if constexpr (FL && D == 3) {
            T preo[D][NPT];
            g2p_block_load<T, D, NPT, NT>(g, gvo, at.tile, tid, preo);
#pragma unroll
            for (int p = 0; p < NPT; ++p) {
                const int i = tid + p * NT;
                if (i < NB)
#pragma unroll
                    for (int a = 0; a < D; ++a) s_vo[a][i] = preo[a][p];
            }
        }
        if constexpr (D == 3)
#pragma unroll
        for (int p = 0; p < NPT; ++p) {
            const int i = tid + p * NT;
            if (i < NB)
#pragma unroll
                for (int a = 0; a < D; ++a) s_v[a][i] = pre[a][p];
        }
        __syncthreads();
        int enn = -1, next2_tile = 0;
        if (!PF) {
            enn = BYTILE ? -1 : __builtin_amdgcn_readfirstlane(tile_entry(it + 2, n_active));
        } else if (en >= 0) {
            g2p_block_load<T, D, NPT, NT>(g, gv, next_tile, tid, pre);
            enn = __builtin_amdgcn_readfirstlane(tile_entry(it + 2, n_active));
            if (enn >= 0) next2_tile = active[enn].tile;
        }
        int tc[3];
        tile_coords(g, at.tile, tc);
        for (int k0 = 0; k0 < at.cnt; k0 += NT) {
            int k = k0 + tid;
            bool valid = k < at.cnt;
            int newkey = 0;
            bool far = false;   // beyond the neighbouring tiles
            if (valid) {
                long long s = at.off + k;
                const bool mine_first = D == 2 && k0 == 0;
                int j = mine_first ? j_first : ld_once(&perm[s]);
                T xp[D];
                AxisFactors<T, D> A;
                int n0 = 0;
                const int stride[3] = {1, BE, BE * BE};
#pragma unroll
                for (int a = 0; a < D; ++a) {
                    xp[a] = mine_first ? x_first[a] : ld_once(&cur.x[a * cap + j]);
                    const T t = mul_exact(xp[a], P.inv), fb = floor(t - T(0.5));
                    A.set(a, t - fb, P.inv, P.h);
                    int l = (int)fb + g.G - tc[a] * TE;
                    l = l < 0 ? 0 : (l > TE - 1 ? TE - 1 : l);   // memory guard only
                    n0 += l * stride[a];
                }
                // vn = sum phi v,  Bm = sum phi v (x_i - x_p)^T,  Lm = sum v (grad phi)^T
                T vn[D], Bm[D][D], Lm[D][D], vo[FL ? D : 1];
#pragma unroll
                for (int a = 0; a < D; ++a) {
                    T R[D][3];
                    axis_sums<DenseBlock<D>>(s_v[a], n0, A, R);
                    vn[a] = dot3(A.w[0], R[0]);
#pragma unroll
                    for (int b = 0; b < D; ++b) {
                        Bm[a][b] = dot3(A.wd[b], R[b]);
                        Lm[a][b] = dot3(A.dw[b], R[b]);
                    }
                    if constexpr (FL) {
                        axis_sums<DenseBlock<D>>(s_vo[a], n0, A, R);
                        vo[a] = dot3(A.w[0], R[0]);
                    }
                }
                bool bad = false, fast = false, noconv = false;
                T xn[D];
#pragma unroll
                for (int a = 0; a < D; ++a) {
                    T xv = xp[a] + P.dt * vn[a];
                    bad |= !finite(xv) || !finite(vn[a]);
                    fast |= fabs(P.dt * vn[a]) > P.h;   // moved more than a cell: CFL violated
                    xv = fmin(fmax(xv, T(0)), P.ext[a]);
                    xn[a] = xv;
                    nxt.x[a * cap + s] = xv;
                    if constexpr (FL) {
                        const T vf = vn[a] + P.flip_alpha * (cur.v[a * cap + j] - vo[a]);
                        bad |= !finite(vf);
                        nxt.v[a * cap + s] = vf;
#pragma unroll
                        for (int b = 0; b < D; ++b) nxt.C[(a * D + b) * cap + s] = T(0);
                    } else {
                        nxt.v[a * cap + s] = vn[a];
#pragma unroll
                        for (int b = 0; b < D; ++b) {
                            T cab;
                            if constexpr (XF == XF_APIC) cab = P.Dinv * Bm[a][b];
                            else if constexpr (XF == XF_TPIC) cab = Lm[a][b];
                            else cab = T(0);
                            nxt.C[(a * D + b) * cap + s] = cab;
                        }
                    }
                }
                if constexpr (MAT == MAT_FLUID) {
                    T dJ = mine_first ? g_first[0] : ld_once(&cur.G[j]), si;
                    fluid_update<T, D>(P, Lm, dJ, si);
                    bad |= !finite(si) || !finite(dJ);
                    st_late(dJ, &nxt.G[s]);
                    nxt.S[s] = si;
                } else if constexpr (MAT == MAT_VFLUID || MAT == MAT_JAUMANN) {
                    T dJ = mine_first ? g_first[0] : ld_once(&cur.G[j]), Sv[NS];
                    if constexpr (MAT == MAT_JAUMANN)   // the viscous fluid's stress is a function of J and L
#pragma unroll
                        for (int q = 0; q < NS; ++q) Sv[q] = cur.S[q * cap + j];
                    if constexpr (MAT == MAT_VFLUID) vfluid_update<T, D>(P, Lm, dJ, Sv);
                    else {
                        // equivalent plastic strain (when carried): App. A's increment
                        T de;
                        jaumann_update<T, D>(P, Lm, dJ, Sv, &de);
                        if (eps_out) eps_out[s] = ld_once(&eps_in[j]) + de;
                    }
                    bad |= !finite(dJ);
                    st_late(dJ, &nxt.G[s]);
#pragma unroll
                    for (int q = 0; q < NS; ++q) {
                        bad |= !finite(Sv[q]);
                        nxt.S[q * cap + s] = Sv[q];
                    }
                } else {
                    T Gm[D][D], Sv[NS];
#pragma unroll
                    for (int a = 0; a < D; ++a)
#pragma unroll
                        for (int b = 0; b < D; ++b)
                            Gm[a][b] = mine_first ? g_first[NG > 1 ? a * D + b : 0] : ld_once(&cur.G[(a * D + b) * cap + j]);
                    T dgam;
                    noconv = !hencky_update<T, D>(P, MAT == MAT_SAND, Lm, Gm, Sv, &dgam);
                    // equivalent plastic strain (when carried): sqrt(2/3) |dE_p|
                    if (MAT == MAT_SAND && eps_out) eps_out[s] = ld_once(&eps_in[j]) + T(0.816496580927726) * dgam;
#pragma unroll
                    for (int a = 0; a < D; ++a)
#pragma unroll
                        for (int b = 0; b < D; ++b) st_late(Gm[a][b], &nxt.G[(a * D + b) * cap + s]);
#pragma unroll
                    for (int q = 0; q < NS; ++q) {
                        bad |= !finite(Sv[q]);
                        nxt.S[q * cap + s] = Sv[q];
                    }
                }
                int pid = mine_first ? pid_first : ld_once(&cur.pid[j]);
                st_late(pid, &nxt.pid[s]);
                if (bad) {
                    atomicOr(&status[0], 1);
                    atomicMin(&status[1], pid);
                }
                if (fast) {
                    atomicOr(&status[0], 2);
                    atomicMin(&status[2], pid);
                }
                if (noconv) {
                    atomicOr(&status[0], 4);
                    atomicMin(&status[3], pid);
                }
                newkey = cell_key<T, D>(g, xn, P.inv);
                key_out[s] = newkey;
                if constexpr (BYTILE)
                    if (k < kTileRow) nd.tile_key[at.tile * kTileRow + k] = newkey;
                if ((D == 3 || BYTILE) && (newkey >> 6) != at.tile) {
                    // into another tile: a neighbouring one is told where from
                    // (2-D: it looks at all its neighbours)
                    int nt[3];
                    tile_coords(g, newkey >> 6, nt);
                    const int dx = tc[0] - nt[0], dy = tc[1] - nt[1], dz = tc[2] - nt[2];
                    far = abs(dx) > 1 || abs(dy) > 1 || abs(dz) > 1;
                    if constexpr (D == 3)
                        atomicOr(&moved[newkey >> 6], far ? kFarBit : 1 << ((dz + 1) * 9 + (dy + 1) * 3 + dx + 1));
                }
            }
            int head, len, rank;
            wave_runs(valid ? (newkey >> 6) : -1, valid, head, len, rank);
            if (valid && rank == 0) atomicAdd(&count[newkey >> 6], len);
            // here, past the particle: inside it the exchange cost registers, and
            // G2P of the viscous fluid 75 us for 73
            if (far) Far{moved, g.ntiles}.push(newkey >> 6, at.off + k);
        }
        __syncthreads();
        e = en;
        if (e >= 0) at = active[e];
        en = enn;
        next_tile = next2_tile;
    }
}

// ---------------------------------------------------------------------------
// Small utility kernels
// ---------------------------------------------------------------------------

template <class T>
__global__ void k_fill(T* p, long long n, T v)
{
    long long i = (long long)blockIdx.x * kBlock + threadIdx.x;
    long long stride = (long long)gridDim.x * kBlock;
    for (; i < n; i += stride) p[i] = v;
}

// Particle field copy between the ABI layout (ncomp x N, memory or pid order)
// and the workspace layout (ncomp x cap, memory order), with the stored-form
// conversions: F = I + G, J = 1 + dJ, symmetric S <-> full dim x dim.
enum { CONV_COPY = 0, CONV_ADD_IDENTITY = 1, CONV_ADD_ONE = 2, CONV_SYM = 3, CONV_ISO = 4 };

// Component c of a field in the ABI layout, of the particle in slot s.
template <class T, int D>
__device__ __forceinline__ T field_value(const T* __restrict__ src, long long cap, long long s, int c, int conv)
{
    const int a = c / D, b = c % D;
    switch (conv) {
    case CONV_ADD_IDENTITY: return src[c * cap + s] + ((a == b) ? T(1) : T(0));
    case CONV_ADD_ONE: return src[s] + T(1);
    case CONV_SYM: {
        int q;
        if (D == 3) q = (a == b) ? a : ((a + b == 1) ? 3 : ((a + b == 2) ? 4 : 5));
        else q = (a == b) ? a : 2;
        return src[q * cap + s];
    }
    case CONV_ISO: return (a == b) ? src[s] : T(0);
    default: return src[c * cap + s];
    }
}

template <class T, int D>
__global__ void k_read_field(const T* __restrict__ src, long long cap, const int32_t* __restrict__ pid,
                             long long N, int ncomp, int conv, int by_pid, T* __restrict__ dst)
{
    long long s = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (s >= N) return;
    long long o = by_pid ? pid[s] : s;
    for (int c = 0; c < ncomp; ++c) dst[c * N + o] = field_value<T, D>(src, cap, s, c, conv);
}

template <int Unused = 0>
__global__ void k_inverse_pid(const int32_t* __restrict__ pid, long long N, int32_t* __restrict__ inv)
{
    long long s = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (s < N) inv[pid[s]] = (int32_t)s;
}

// The same in pid order, gathered through the inverse of pid (several
// components: the inverse's scatter is paid once).  Scattering the components
// by pid wrote 8 to 16 bytes of a line at a time from all eight L2s.  Here the
// writes are whole lines; one component per grid row and one contiguous eighth
// of the particles per XCD keep the source lines that neighbouring particles
// share in that XCD's L2.  Cylinder (2,780,000 particles), mean of x, v, C,
// F and the stress: binary32 87 -> 56 + 12 us for the inverse, binary64
// 114 -> 80 + 13; one particle per thread 65, bound by the latency of the two
// dependent loads.
constexpr int kGatherPer = 4;   // particles per thread, loaded together

template <class T, int D>
__global__ __launch_bounds__(kBlock) void k_gather_field(const T* __restrict__ src, long long cap,
                                                         const int32_t* __restrict__ inv, long long N, int conv,
                                                         T* __restrict__ dst)
{
    const long long blk = (long long)(blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
    const long long o0 = blk * (kBlock * kGatherPer) + threadIdx.x;
    const int c = blockIdx.y;
    int at[kGatherPer];
    T v[kGatherPer];
#pragma unroll
    for (int q = 0; q < kGatherPer; ++q) at[q] = o0 + q * kBlock < N ? inv[o0 + q * kBlock] : 0;
#pragma unroll
    for (int q = 0; q < kGatherPer; ++q) v[q] = field_value<T, D>(src, cap, at[q], c, conv);
#pragma unroll
    for (int q = 0; q < kGatherPer; ++q)
        if (o0 + q * kBlock < N) dst[c * N + o0 + q * kBlock] = v[q];
}

template <class T, int D>
__global__ void k_write_field(T* __restrict__ dst, long long cap, const int32_t* __restrict__ pid,
                              long long N, int ncomp, int conv, int by_pid, const T* __restrict__ src)
{
    long long s = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (s >= N) return;
    long long o = by_pid ? pid[s] : s;
    if (conv == CONV_SYM) {
        if (D == 3) {
            dst[0 * cap + s] = src[0 * N + o];
            dst[1 * cap + s] = src[4 * N + o];
            dst[2 * cap + s] = src[8 * N + o];
            dst[3 * cap + s] = T(0.5) * (src[1 * N + o] + src[3 * N + o]);
            dst[4 * cap + s] = T(0.5) * (src[2 * N + o] + src[6 * N + o]);
            dst[5 * cap + s] = T(0.5) * (src[5 * N + o] + src[7 * N + o]);
        } else {
            dst[0 * cap + s] = src[0 * N + o];
            dst[1 * cap + s] = src[3 * N + o];
            dst[2 * cap + s] = T(0.5) * (src[1 * N + o] + src[2 * N + o]);
        }
        return;
    }
    if (conv == CONV_ISO) {
        T tr = T(0);
        for (int a = 0; a < D; ++a) tr += src[(a * D + a) * N + o];
        dst[s] = tr / T(D);
        return;
    }
    for (int c = 0; c < ncomp; ++c) {
        int a = c / D, b = c % D;
        T v = src[c * N + o];
        if (conv == CONV_ADD_IDENTITY) v -= (a == b) ? T(1) : T(0);
        if (conv == CONV_ADD_ONE) v -= T(1);
        dst[c * cap + s] = v;
    }
}

// Dense node box (n + 1 + 2G per axis) from the tile-padded grid.  The grid
// kernel writes only the node blocks of the step's active tiles, so a node
// that no active tile's block covers holds a value of an earlier step; it is
// read as zero (no mass, no velocity), which is what the step's grid holds
// there.  tile_slot[t] >= 0 marks the active tiles of the step.
template <class T>
__global__ void k_read_grid(Geo g, const T* __restrict__ src, int ncomp, const int* __restrict__ tile_slot,
                            T* __restrict__ dst)
{
    long long nbox = (long long)g.box[0] * g.box[1] * g.box[2];
    long long i = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (i >= nbox) return;
    int I[3];
    I[0] = (int)(i % g.box[0]);
    long long r = i / g.box[0];
    I[1] = (int)(r % g.box[1]);
    I[2] = (int)(r / g.box[1]);
    // tiles whose (T+2)-node block holds the node: own = I / T, and own - 1
    // where I lies in the first two nodes of its tile
    int lo[3], hi[3];
    for (int a = 0; a < 3; ++a) {
        int own = (a < g.dim) ? I[a] / g.T : 0;
        hi[a] = own;
        lo[a] = (a < g.dim && I[a] % g.T < 2 && own >= 1) ? own - 1 : own;
    }
    bool live = false;
    for (int tz = lo[2]; tz <= hi[2]; ++tz)
        for (int ty = lo[1]; ty <= hi[1]; ++ty)
            for (int tx = lo[0]; tx <= hi[0]; ++tx)
                live |= tile_slot[((long long)tz * g.ntile[1] + ty) * g.ntile[0] + tx] >= 0;
    long long node = node_index(g, I[0], I[1], I[2]);
    for (int c = 0; c < ncomp; ++c) dst[c * nbox + i] = live ? src[c * g.NN + node] : T(0);
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

// Whether a read in pid order gathers (two launches), or scatters the
// components of each slot.  3-D matrices gather from 2.5 M values on: below, the
// second launch costs more than the scattered lines, which then stay in cache
// (lattice order, 9 components, scatter and gather 6.8 and 10.2 us at 110,592
// particles, 10.9 and 10.9 at 262,144, 161 and 115 at 2,935,296).  3-D vectors
// are scattered as fast while they fit the cache, and again far past it: binary32
// 45.9 and 49.9 us at 35 MB, 77 and 84 at 64 MB, 329 and 235 at 129 MB; binary64
// 20.3 and 21.8 at 20 MB, 37.6 and 36.6 at 42 MB, 59 and 57 at 70 MB, 205 and 145 at
// 127 MB, 310 and 323 at 258 MB.  In 2-D a
// tile's rows are eight cells long and the scatter is the faster at every size
// (binary32, 2.5 M particles, vectors 18.6 and 26.3 us, matrices 31.2 and 39.1;
// 6.0 M binary64, 56 and 60, 152 and 156).
inline bool read_gathers(int dim, long long N, int ncomp, int elem)
{
    const long long values = N * ncomp, bytes = values * elem;
    return dim == 3 && (ncomp == 9 ? values >= 2500000 : ncomp == 3 && bytes > (elem == 8 ? 40000000 : 100000000) && bytes < 200000000);
}

inline unsigned nblocks(long long n) { return (unsigned)((n + kBlock - 1) / kBlock); }

template <class T>
Phys<T> make_phys(const mpm_ctx* c, double dt)
{
    Phys<T> P{};
    const mpm_config& k = c->cfg;
    int D = k.dim;
    P.h = (T)k.dx;
    P.inv = T(1) / (T)k.dx;
    P.Dinv = T(4) / ((T)k.dx * (T)k.dx);
    P.dt = (T)dt;
    P.mass = (T)c->mass;
    P.vol0 = (T)c->vol0;
    for (int a = 0; a < 3; ++a) {
        P.g[a] = (T)k.gravity[a];
        P.ext[a] = (a < D) ? (T)((double)k.n[a] * k.dx) : T(0);
    }
    double E = k.youngs, nu = k.poisson;
    double lam = E * nu / ((1.0 + nu) * (1.0 - 2.0 * nu));
    double mu = E / (2.0 * (1.0 + nu));
    double s = sin(k.phi_deg * M_PI / 180.0);
    double q_phi = 6.0 * s / (sqrt(3.0) * (3.0 + s));
    double alpha = sqrt(2.0) / 3.0 * q_phi;
    P.lam = (T)lam;
    P.mu = (T)mu;
    P.cone_coef = (T)((D * lam + 2.0 * mu) / (2.0 * mu) * alpha);
    P.k_over_gamma = (T)(k.bulk / k.gamma);
    P.gamma = (T)k.gamma;
    P.material = c->mat;
    for (int f = 0; f < 6; ++f) {
        P.wall_mode[f] = k.wall_mode[f];
        P.wall_mu[f] = (T)k.wall_mu[f];
    }
    P.floor_mu = (const T*)c->floor_mu;
    P.floor_stride = c->geo.box[0];
    P.keep_grid = k.keep_grid;
    P.xfer = c->xfer;
    P.flip_alpha = (T)k.flip_alpha;
    P.visc = (T)k.viscosity;
    {
        // hypoelastic Drucker-Prager constants (App. A)
        double sp = sin(k.phi_deg * M_PI / 180.0), cp = cos(k.phi_deg * M_PI / 180.0);
        double ss = sin(k.psi_deg * M_PI / 180.0);
        double q_phi = 6.0 * sp / (sqrt(3.0) * (3.0 + sp));
        double k_phi = 6.0 * k.cohesion * cp / (sqrt(3.0) * (3.0 + sp));
        double q_psi = 6.0 * ss / (sqrt(3.0) * (3.0 + ss));
        P.jK = (T)(lam + 2.0 * mu / D);
        P.jq_phi = (T)q_phi;
        P.jk_phi = (T)k_phi;
        P.jq_psi = (T)q_psi;
        P.jst = (T)k.tension;
        P.jtauP = (T)(k_phi - q_phi * k.tension);
        P.jalphaP = (T)(sqrt(1.0 + q_phi * q_phi) - q_phi);
        P.jband2 = (T)(1e-6 * E * 1e-6 * E);
    }
    P.n_obst = k.n_obstacles;
    P.obst_h = k.dx;
    for (int o = 0; o < kMaxObstacles; ++o) {
        int ok = 0;
        for (int a = 0; a < 3; ++a) {
            P.obst_lo[o][a] = k.obst_lo[o][a];
            P.obst_hi[o][a] = k.obst_hi[o][a];
            if (a < D) {
                double ext = (double)k.n[a] * k.dx;
                if (k.obst_lo[o][a] > 0.0) ok |= 1 << (2 * a);        // lower face inside the domain
                if (k.obst_hi[o][a] < ext) ok |= 1 << (2 * a + 1);    // upper face inside the domain
            }
        }
        P.obst_face_ok[o] = ok;
    }
    return P;
}

template <class T>
PView<T> view(const mpm_ctx* c, int which)
{
    PView<T> v{};
    T* base = (T*)c->st[which];
    long long cap = c->cap;
    int D = c->cfg.dim;
    v.cap = cap;
    v.x = base;
    v.v = base + D * cap;
    v.C = base + 2 * D * cap;
    v.G = base + (2 * D + D * D) * cap;
    v.S = v.G + (mat_has_F(c->mat) ? D * D : 1) * cap;
    v.pid = c->pid[which];
    return v;
}

// Workgroups of a per-tile launch with `block` threads each: enough to fill the
// chip, and not more than the grid has tiles (a small grid's launch was 2048
// workgroups for a few dozen tiles).  A multiple of 8, one share per XCD.
inline unsigned tile_wgs(const mpm_ctx* c, int block)
{
    const long long full = (long long)kTileWGs * kBlock / block, tiles = (c->geo.ntiles + 7) / 8 * 8;
    return (unsigned)std::min(full, (long long)tiles);
}

// Whether P2G reads the particles with the non-temporal hint.  A tile's waves
// read the same lines, so caching pays where the state that G2P has just written
// is still in the 256 MB cache: P2G on the cylinder, plain and hinted, 42 MB
// 15.8 and 17.4 us, 112 MB 29.7 and 36.1, 198 MB 43.5 and 47.2 (the step 181.0
// both: the other kernels lose what P2G gains); past it the hint keeps the lines
// that the grid update and G2P need: the step 265.4 and 263.2 us at 334 MB, 328
// and 314 at 396 MB (binary64), 484 and 463 at 667 MB.  With FLIP four waves
// read them and plain is better at every size (617 and 616 us at 667 MB, 332
// and 336 at 334 MB, 142 and 154 at 112 MB).  Where no step has laid out the
// particles, those of a tile lie apart and share their lines with many other
// tiles': hinted, each of them fetches the line again.  2.94 M particles from a
// lattice, first step, P2G hinted and plain: sand binary32 977 and 573 us, binary64
// 1256 and 699, fluid binary64 954 and 449.
inline bool p2g_hint(const mpm_ctx* c, bool laid_out) { return laid_out && (double)c->nsc * (double)c->cap * c->elem > 200e6; }

template <class T, int D>
struct Solver {
    static int launch_err(mpm_ctx* c, const char* what) { return hip_check(c, hipGetLastError(), what); }

    static int init_particles(mpm_ctx* c, const void* x, const void* v)
    {
        match_turn(c, false);
        clear_keys(c);
        if (c->cap > 0)
            k_init<T, D><<<nblocks(c->cap), kBlock, 0, c->stream>>>(
                c->geo, make_phys<T>(c, 0.0), (const T*)x, (const T*)v, c->N, view<T>(c, c->cur), c->nsc, (T*)c->eps[0],
                (T*)c->eps[1], c->key, key_count(c));
        return launch_err(c, "init particles");
    }

    static int recompute_keys(mpm_ctx* c)
    {
        match_turn(c, false);
        new_keys(c, view<T>(c, c->cur));
        return launch_err(c, "keys");
    }

    // Whether steps alternate between two sets of ranges (2-D: and counts).
    static bool alternates(const mpm_ctx* c) { return D == 3 || c->geo.ntiles <= kSmallTiles; }
    // Between calls the set in use goes with the state buffer in use, so that
    // captured steps find both where they were at the capture whenever the
    // state is in the same buffer again.  carry: the set's contents move.
    static void match_turn(mpm_ctx* c, bool carry)
    {
        if (!alternates(c) || c->turn == c->cur) return;
        if (carry) {
            const int n = c->geo.ntiles;
            k_copy_layout<0><<<std::min<long long>(nblocks(n), 4096), kBlock, 0, c->stream>>>(
                c->range[c->turn], c->range[c->cur], D == 2 ? c->count[c->turn] : nullptr, c->count[D == 2 ? c->cur : 0], n);
        }
        c->turn = c->cur;
    }

    static int* key_count(const mpm_ctx* c) { return c->count[D == 2 ? c->turn : 0]; }
    // No step has laid out the state that follows.
    static void clear_keys(mpm_ctx* c)
    {
        k_clear_keys<0><<<std::min<long long>(nblocks(c->geo.ntiles), 4096), kBlock, 0, c->stream>>>(
            key_count(c), Far{c->moved, c->geo.ntiles}, c->geo.ntiles);
        c->ranges_known = false;
    }

    // Keys and tile counts of a state whose layout no sort of this step's
    // predecessor describes.
    static void new_keys(mpm_ctx* c, const PView<T>& v)
    {
        clear_keys(c);
        if (c->N > 0) {
            Phys<T> P = make_phys<T>(c, 0.0);
            k_keys<T, D><<<nblocks(c->N), kBlock, 0, c->stream>>>(c->geo, P, v, c->N, c->key, key_count(c));
        }
    }

    static int clear_grid(mpm_ctx* c)
    {
        hipStream_t st = c->stream;
        long long NN = c->geo.NN;
        k_fill<T><<<4096, kBlock, 0, st>>>((T*)c->gv, D * NN, T(0));
        k_fill<T><<<4096, kBlock, 0, st>>>((T*)c->gmass, NN, T(0));
        if (c->gvo) k_fill<T><<<4096, kBlock, 0, st>>>((T*)c->gvo, D * NN, T(0));
        k_fill<int><<<1, kBlock, 0, st>>>(c->status, 16, 0);
        k_fill<int><<<1, kBlock, 0, st>>>(c->status + 1, 3, 0x7fffffff);
        if (c->geo.ntiles > 0)
            k_fill<int><<<std::min<long long>(nblocks(c->geo.ntiles), 4096), kBlock, 0, st>>>(c->tile_slot, c->geo.ntiles, -1);
        if (D == 3) k_fill<int><<<1, kBlock, 0, st>>>(c->meta, 64, 0);
        clear_keys(c);
        return launch_err(c, "clear grid");
    }

    // Where one step keeps its sort and grid: the context's own arrays, or a
    // record of the grid tape (then the nodal velocity before the walls is
    // kept too, for the adjoint).
    struct StepBufs {
        int32_t* perm;
        int32_t* tile_slot;
        ActiveTile* active;
        int32_t* meta;
        T* gv;
        T* gmass;
        T* gvt;
        T* gvo;     // FLIP: nodal velocity before the update
        const T* eps_in = nullptr;   // equivalent plastic strain, when carried
        T* eps_out = nullptr;
    };
    static StepBufs ctx_bufs(mpm_ctx* c)
    {
        // in 2-D G2P forms the velocity before the update itself: only the reverse sweep reads it
        return {c->perm, c->tile_slot, c->active, c->meta, (T*)c->gv, (T*)c->gmass, nullptr, D == 2 ? nullptr : (T*)c->gvo};
    }

    // One step from state view cur into state view nxt with the transfer XF
    // (FLIP: P2G and the grid update also form the velocity before the
    // update).  The transfer is a template parameter: as a run-time choice it
    // kept both affine candidates live in G2P and cost it half its waves.
    // Without `advance` the new particle state is not wanted: in 3-D the step
    // ends with the grid (in 2-D the nodes are formed by G2P's launch), and the
    // caller forms the keys before the next step (new_keys).
    template <int MAT, int XF = XF_APIC>
    static void step_views(mpm_ctx* c, const Phys<T>& P, const PView<T>& cur, const PView<T>& nxt,
                           const StepBufs& b, bool advance = true)
    {
        constexpr bool FL = XF == XF_FLIP;
        // P2G depends on the material only through the stored stress: one
        // isotropic value or the symmetric tensor
        constexpr int PM = mat_iso_stress(MAT) ? MAT_FLUID : MAT_SAND;
        hipStream_t st = c->stream;
        const Geo& g = c->geo;
        unsigned nsb = (unsigned)((g.ntiles + kScanChunk - 1) / kScanChunk);
        const unsigned long long seq = work_seq(c);
        prof_mark(c, -1);
        if constexpr (D == 2) {
            step_views2<MAT, XF>(c, P, cur, nxt, b, nsb, seq);
            return;
        } else {
        const int o = c->turn, n = 1 - o;
        int* count = c->count[0];
        const Ranges r{count, nullptr, c->range[o], c->range[n], c->moved, c->key, nullptr, nullptr, (long long)c->N};
        scan_tiles(c, nsb, count, b, c->range[n], nullptr);
        const unsigned swgs = tile_wgs(c, kSortBlock);
        const bool gather = know_ranges(c, seq) && c->N < (1ll << 30);   // key positions plus a batch stay in int32
        if (gather) {
            k_sort_gather<0><<<swgs, kSortBlock, 0, st>>>(g, r, b.meta, c->meta + kHaloSum, b.active, c->tmp, c->tmpk, b.perm, c->cell_cnt);
        } else {
            bucket(c, count);
            k_sort<0><<<swgs, kSortBlock, 0, st>>>(Far{c->moved, g.ntiles}, b.meta, c->meta + kHaloSum, b.active, c->tmp, c->tmpk, b.perm, c->cell_cnt);
        }
        prof_mark(c, MPM_PROF_BUCKET);
        if (!FL && p2g_hint(c, gather))
            k_p2g<T, D, PM, FL, !FL><<<tile_wgs(c, kP2GBlock<FL>), kP2GBlock<FL>, 0, st>>>(g, P, b.meta, b.active, c->cell_cnt,
                                                                                        cur, b.perm, (T*)c->part_grid);
        else
            k_p2g<T, D, PM, FL, false><<<tile_wgs(c, kP2GBlock<FL>), kP2GBlock<FL>, 0, st>>>(g, P, b.meta, b.active, c->cell_cnt,
                                                                                         cur, b.perm, (T*)c->part_grid);
        prof_mark(c, MPM_PROF_P2G);
        k_grid<T, D, FL><<<tile_wgs(c, kGridBlock), kGridBlock, 0, st>>>(g, P, b.meta, b.active, b.tile_slot, (const T*)c->part_grid,
                                                  b.gv, b.gmass, b.gvt, b.gvo);
        prof_mark(c, MPM_PROF_GRID);
        if (advance) {
            k_g2p<T, D, MAT, XF, false><<<tile_wgs(c, kG2PBlock<T, D>), kG2PBlock<T, D>, 0, st>>>(g, P, b.meta, b.active, b.perm, cur, nxt, (const T*)b.gv,
                                                          (const T*)b.gvo, c->key, count, c->status, b.eps_in, b.eps_out, Nodes2<T>{}, c->moved);
            prof_mark(c, MPM_PROF_G2P);
        }
        c->turn = n;
        c->ranges_known = true;
        c->ranges_seq = seq;
        }
    }

    // The scan over the tiles' counts.
    static void scan_tiles(mpm_ctx* c, unsigned nsb, const int* count, const StepBufs& b, int2* range, int* count_next)
    {
        hipStream_t st = c->stream;
        const Geo& g = c->geo;
        const Halo halo{D == 3 ? c->meta + kHaloSum : nullptr, g.ntile[0], g.ntile[1], (int)nsb};
        const bool once = g.ntiles <= kScanOnceTiles;
        // the list's workgroups: a tile per thread, as far as the chip has room
        const int nt = once ? kScanOnce : kBlock;
        const unsigned wgs = nsb + (D == 3 ? (unsigned)std::min((g.ntiles + nt - 1) / nt, 1024) : 0u);
        if (once) {
            k_scan_once<0><<<wgs, kScanOnce, 0, st>>>(count, g.ntiles, c->tile_off, b.tile_slot, b.active, b.meta, range,
                                                      count_next, halo);
        } else {
            k_scan_reduce<0><<<nsb, kBlock, 0, st>>>(count, g.ntiles, c->part);
            k_scan_down<0><<<wgs, kBlock, 0, st>>>(count, g.ntiles, c->part, c->tile_off, b.tile_slot, b.active, b.meta, range,
                                                   count_next, halo);
        }
        prof_mark(c, MPM_PROF_SCAN);
    }

    // The scatter of the particles into their tiles' ranges (clears the counts).
    static void bucket(mpm_ctx* c, int* count)
    {
        k_bucket<0><<<(unsigned)((c->N + kBlock * kBucketPer - 1) / (kBlock * kBucketPer)), kBlock, 0, c->stream>>>(
            c->N, c->key, count, c->tile_off, c->tmp, c->tmpk);
    }

    // The step in 2-D: two launches where the last sort's layout is known and
    // the tiles are few enough that a workgroup can sum all earlier counts
    // itself (one scan chunk: 8 loads per thread), else the scan and the
    // scatter before them.  Everything that alternates between steps does so on
    // every step, so that an even number of captured steps can be replayed (the
    // first of them finds its particles by their keys, see work_seq).
    template <int MAT, int XF>
    static void step_views2(mpm_ctx* c, const Phys<T>& P, const PView<T>& cur, const PView<T>& nxt, const StepBufs& b,
                            unsigned nsb, unsigned long long seq)
    {
        constexpr bool FL = XF == XF_FLIP;
        constexpr int PM = mat_iso_stress(MAT) ? MAT_FLUID : MAT_SAND;
        hipStream_t st = c->stream;
        const Geo& g = c->geo;
        const bool small = g.ntiles <= kSmallTiles, narrow = sizeof(T) == 8 && c->N > kNarrow2;
        const int o = c->turn, n = small ? 1 - o : o;
        const unsigned wgs = small ? (unsigned)((g.ntiles + 7) / 8 * 8) : (unsigned)kTileWGs;
        const Ranges r{c->count[o], c->count[n], c->range[o], c->range[n], c->moved, c->key, c->tile_key,
                          small ? c->tile_perm : nullptr, (long long)c->N};
        if (small && know_ranges(c, seq) && c->N < (1ll << 30)) {   // key positions plus a batch stay in int32
            k_sort_p2g2<T, PM, FL, true, 256><<<wgs, 256, 0, st>>>(g, P, r, b.meta, b.active, b.tile_slot, c->tmp, c->tmpk,
                                                                      cur, b.perm, (T*)c->part_grid);
        } else {
            scan_tiles(c, nsb, c->count[o], b, small ? c->range[n] : nullptr, small ? c->count[n] : nullptr);
            bucket(c, c->count[o]);
            prof_mark(c, MPM_PROF_BUCKET);
            if (small)
                k_sort_p2g2<T, PM, FL, false, 256><<<wgs, 256, 0, st>>>(g, P, r, b.meta, b.active, b.tile_slot, c->tmp,
                                                                        c->tmpk, cur, b.perm, (T*)c->part_grid);
            else if (narrow)
                k_sort_p2g2<T, PM, FL, false, kSortNarrow2<T>><<<tile_wgs(c, kSortNarrow2<T>), kSortNarrow2<T>, 0, st>>>(
                    g, P, r, b.meta, b.active, b.tile_slot, c->tmp, c->tmpk, cur, b.perm, (T*)c->part_grid);
            else
                k_sort_p2g2<T, PM, FL, false, kSortMany2><<<tile_wgs(c, kSortMany2), kSortMany2, 0, st>>>(
                    g, P, r, b.meta, b.active, b.tile_slot, c->tmp, c->tmpk, cur, b.perm, (T*)c->part_grid);
        }
        prof_mark(c, MPM_PROF_P2G);
        const Nodes2<T> nd{(const T*)c->part_grid, b.tile_slot, small ? c->range[n] : nullptr, c->tile_perm, c->tile_key, b.gv, b.gmass, b.gvt, b.gvo};
        auto g2p = [&](auto* kernel, unsigned grid, int block) {
            kernel<<<grid, block, 0, st>>>(g, P, b.meta, b.active, b.perm, cur, nxt, nullptr, nullptr, c->key, c->count[n], c->status,
                                           b.eps_in, b.eps_out, nd, c->moved);
        };
        if (small) g2p(k_g2p<T, D, MAT, XF, true>, wgs, kG2PBlock<T, D>);
        else if (narrow) g2p(k_g2p<T, D, MAT, XF, false, kG2PNarrow2<T>>, tile_wgs(c, kG2PNarrow2<T>), kG2PNarrow2<T>);
        else g2p(k_g2p<T, D, MAT, XF, false>, wgs, kG2PBlock<T, D>);
        prof_mark(c, MPM_PROF_G2P);
        c->turn = n;
        c->ranges_known = small;
        c->ranges_seq = seq;
    }

    template <int MAT, int XF = XF_APIC>
    static void step_views(mpm_ctx* c, const Phys<T>& P, const PView<T>& cur, const PView<T>& nxt)
    {
        step_views<MAT, XF>(c, P, cur, nxt, ctx_bufs(c));
    }

    template <int MAT, int XF>
    static void one_step(mpm_ctx* c, const Phys<T>& P)
    {
        StepBufs b = ctx_bufs(c);
        if ((MAT == MAT_SAND || MAT == MAT_JAUMANN) && c->eps[0]) {
            b.eps_in = (const T*)c->eps[c->cur];
            b.eps_out = (T*)c->eps[1 - c->cur];
        }
        step_views<MAT, XF>(c, P, view<T>(c, c->cur), view<T>(c, 1 - c->cur), b);
        c->cur = 1 - c->cur;
    }

    template <int XF>
    static void one_step_x(mpm_ctx* c, const Phys<T>& P)
    {
        switch (c->mat) {
        case MAT_FLUID: one_step<MAT_FLUID, XF>(c, P); break;
        case MAT_SAND: one_step<MAT_SAND, XF>(c, P); break;
        case MAT_VFLUID: one_step<MAT_VFLUID, XF>(c, P); break;
        case MAT_JAUMANN: one_step<MAT_JAUMANN, XF>(c, P); break;
        default: one_step<MAT_ELASTIC, XF>(c, P); break;
        }
    }

    static int step(mpm_ctx* c, int n, double dt)
    {
        Phys<T> P = make_phys<T>(c, dt);
        for (int i = 0; i < n; ++i) {
            switch (c->xfer) {
            case XF_PIC: one_step_x<XF_PIC>(c, P); break;
            case XF_FLIP: one_step_x<XF_FLIP>(c, P); break;
            case XF_TPIC: one_step_x<XF_TPIC>(c, P); break;
            default: one_step_x<XF_APIC>(c, P); break;
            }
        }
        return launch_err(c, "step");
    }

    // field -> (pointer into state, ncomp in ABI layout, conversion)
    static int field_desc(mpm_ctx* c, int field, T** ptr, int* ncomp, int* conv)
    {
        PView<T> s = view<T>(c, c->cur);
        const bool fluid = !mat_has_F(c->mat);   // carries J instead of F
        const bool iso = mat_iso_stress(c->mat);
        switch (field) {
        case MPM_FIELD_X: *ptr = s.x; *ncomp = D; *conv = CONV_COPY; return MPM_OK;
        case MPM_FIELD_V: *ptr = s.v; *ncomp = D; *conv = CONV_COPY; return MPM_OK;
        case MPM_FIELD_C: *ptr = s.C; *ncomp = D * D; *conv = CONV_COPY; return MPM_OK;
        case MPM_FIELD_F:
            if (fluid) break;
            *ptr = s.G; *ncomp = D * D; *conv = CONV_ADD_IDENTITY; return MPM_OK;
        case MPM_FIELD_FMI:
            if (fluid) break;
            *ptr = s.G; *ncomp = D * D; *conv = CONV_COPY; return MPM_OK;
        case MPM_FIELD_J:
            if (!fluid) break;
            *ptr = s.G; *ncomp = 1; *conv = CONV_ADD_ONE; return MPM_OK;
        case MPM_FIELD_JM1:
            if (!fluid) break;
            *ptr = s.G; *ncomp = 1; *conv = CONV_COPY; return MPM_OK;
        case MPM_FIELD_STRESS:
            *ptr = s.S; *ncomp = D * D; *conv = iso ? CONV_ISO : CONV_SYM; return MPM_OK;
        case MPM_FIELD_EPS_EQ:
            if (!c->eps[c->cur]) return set_err(c, MPM_EINVAL, "EPS_EQ needs track_eps_eq = 1");
            *ptr = (T*)c->eps[c->cur]; *ncomp = 1; *conv = CONV_COPY; return MPM_OK;
        default: break;
        }
        return set_err(c, MPM_EINVAL, "field not available for this material");
    }

    static int read_state(mpm_ctx* c, int field, int order, void* dst)
    {
        hipStream_t st = c->stream;
        PView<T> s = view<T>(c, c->cur);
        long long N = c->N;
        if (field == MPM_FIELD_PID) {
            if (order == MPM_ORDER_PID) return set_err(c, MPM_EINVAL, "pid in pid order is the identity");
            if (hipMemcpyAsync(dst, s.pid, sizeof(int32_t) * N, hipMemcpyDeviceToDevice, st) != hipSuccess)
                return launch_err(c, "read pid");
            return MPM_OK;
        }
        T* src;
        int ncomp, conv;
        int rc = field_desc(c, field, &src, &ncomp, &conv);
        if (rc) return rc;
        if (order == MPM_ORDER_PID && read_gathers(D, N, ncomp, (int)sizeof(T))) {
            k_inverse_pid<0><<<nblocks(N), kBlock, 0, st>>>(s.pid, N, c->inv);
            k_gather_field<T, D><<<dim3((nblocks(N) + 8 * kGatherPer - 1) / (8 * kGatherPer) * 8, ncomp), kBlock, 0, st>>>(src, c->cap, c->inv, N, conv,
                                                                                          (T*)dst);
        } else if (N > 0) {
            k_read_field<T, D><<<nblocks(N), kBlock, 0, st>>>(src, c->cap, s.pid, N, ncomp, conv,
                                                             order == MPM_ORDER_PID, (T*)dst);
        }
        return launch_err(c, "read state");
    }

    static int write_state(mpm_ctx* c, int field, int order, const void* src)
    {
        hipStream_t st = c->stream;
        PView<T> s = view<T>(c, c->cur);
        long long N = c->N;
        if (field == MPM_FIELD_PID) return set_err(c, MPM_EINVAL, "pid cannot be written");
        T* dstp;
        int ncomp, conv;
        int rc = field_desc(c, field, &dstp, &ncomp, &conv);
        if (rc) return rc;
        if (N > 0)
            k_write_field<T, D><<<nblocks(N), kBlock, 0, st>>>(dstp, c->cap, s.pid, N, ncomp, conv,
                                                              order == MPM_ORDER_PID, (const T*)src);
        rc = launch_err(c, "write state");
        if (rc) return rc;
        if (field == MPM_FIELD_X) return recompute_keys(c);
        return MPM_OK;
    }

    static int read_grid(mpm_ctx* c, int which, void* dst)
    {
        const Geo& g = c->geo;
        long long nbox = (long long)g.box[0] * g.box[1] * g.box[2];
        if (which == MPM_GRID_MASS) {
            if (!c->cfg.keep_grid) return set_err(c, MPM_EINVAL, "grid mass needs keep_grid = 1");
            k_read_grid<T><<<nblocks(nbox), kBlock, 0, c->stream>>>(g, (const T*)c->gmass, 1, c->tile_slot, (T*)dst);
        } else if (which == MPM_GRID_VEL) {
            k_read_grid<T><<<nblocks(nbox), kBlock, 0, c->stream>>>(g, (const T*)c->gv, D, c->tile_slot, (T*)dst);
        } else {
            return set_err(c, MPM_EINVAL, "unknown grid field");
        }
        return launch_err(c, "read grid");
    }

    static Ops table()
    {
        Ops o;
        o.init_particles = &init_particles;
        o.recompute_keys = &recompute_keys;
        o.clear_grid = &clear_grid;
        o.step = &step;
        o.read_state = &read_state;
        o.write_state = &write_state;
        o.read_grid = &read_grid;
        return o;
    }
};

}  // namespace mpm
