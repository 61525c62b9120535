// Particle <-> mesh kernels (Sec. 2 of Angus et al.): cloud-in-cell mass
// assignment in 64-bit fixed point (step 1), the Eq. 1 right-hand side, and
// the force gather with the same cloud-in-cell weights, plus the circular
// speed of Eq. 4.
//
// The deposit's weights are plain IEEE products (no fused multiply-add) and
// each corner receives rint(w m 2^s) as a 64-bit integer, so the integer grid
// does not depend on the order in which atomics land.
#include "common.h"

namespace qm {

// ------------------------------------------------------------------ deposit
//
// Workgroup g takes a contiguous share of the particles.  For each box it
// clears an LDS window of kWin nodes around the box centre, adds every corner
// of the particles whose whole cloud lies in the window with LDS 64-bit
// atomics, sends the other particles' corners to the grid with global 64-bit
// atomics, and writes the window to its scratch slab.  A second kernel sums
// the slabs of all workgroups into the grid.  Integer addition makes the
// result independent of the order of every add.

__device__ __forceinline__ bool cic_cell(const BoxGeom &g, int n, double px, double py, double pz, int ic[3],
                                         double w[3][2])
{
#pragma clang fp contract(off)
    const double top = (double)(n - 1);
    const double ux = (px - g.xmin) * g.inv_h;
    const double uy = (py - g.xmin) * g.inv_h;
    const double uz = (pz - g.xmin) * g.inv_h;
    if (!(ux >= 0.0 && ux < top && uy >= 0.0 && uy < top && uz >= 0.0 && uz < top)) return false;
    const double fx0 = floor(ux), fy0 = floor(uy), fz0 = floor(uz);
    ic[0] = (int)fx0;
    ic[1] = (int)fy0;
    ic[2] = (int)fz0;
    const double fx = ux - fx0, fy = uy - fy0, fz = uz - fz0;
    w[0][0] = 1.0 - fx;
    w[0][1] = fx;
    w[1][0] = 1.0 - fy;
    w[1][1] = fy;
    w[2][0] = 1.0 - fz;
    w[2][1] = fz;
    return true;
}

// A workgroup's share; W and cnt_sh: LDS.
__device__ __forceinline__ void window_share(const DepositArgs &A, const double *__restrict__ x,
                                             const double *__restrict__ y, const double *__restrict__ z,
                                             const double *__restrict__ m, int64_t np, int64_t per_block,
                                             unsigned long long *__restrict__ inside_count,
                                             unsigned long long (&W)[kWin], unsigned int &cnt_sh)
{
#pragma clang fp contract(off)
    const int64_t p0 = (int64_t)blockIdx.x * per_block;
    const int64_t p1 = min(np, p0 + per_block);
    if (threadIdx.x == 0) cnt_sh = 0;
    unsigned int in0 = 0;
    for (int b = 0; b < A.nbox; ++b) {
        for (int e = threadIdx.x; e < kWin; e += kDepositThreads) W[e] = 0ULL;
        __syncthreads();
        const BoxGeom g = A.box[b];
        const int wx = A.w0[b][0], wy = A.w0[b][1], wz = A.w0[b][2];
        unsigned long long *q = A.q[b];
        for (int64_t p = p0 + threadIdx.x; p < p1; p += kDepositThreads) {
            int ic[3];
            double w[3][2];
            if (!cic_cell(g, A.n, x[p], y[p], z[p], ic, w)) continue;
            if (b == 0) ++in0;
            const double pm = m[p];
            const int lx = ic[0] - wx, ly = ic[1] - wy, lz = ic[2] - wz;
            const bool inwin = lx >= 0 && lx < kWinX - 1 && ly >= 0 && ly < kWinY - 1 && lz >= 0 && lz < kWinZ - 1;
            for (int c = 0; c < 2; ++c)
                for (int bb = 0; bb < 2; ++bb)
                    for (int a = 0; a < 2; ++a) {
                        const double wt = (w[0][a] * w[1][bb]) * w[2][c];
                        const unsigned long long qv = (unsigned long long)__double2ll_rn((wt * pm) * A.scale);
                        // a scope of its own keeps the two apart: of one, they became one flat atomic
                        if (inwin)
                            __hip_atomic_fetch_add(&W[(lx + a) + kWinX * ((ly + bb) + kWinY * (lz + c))], qv,
                                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        else
                            atomicAdd(q + id3(A.n, ic[0] + a, ic[1] + bb, ic[2] + c), qv);
                    }
        }
        __syncthreads();
        unsigned long long *slab = A.scratch + ((size_t)blockIdx.x * A.nbox + b) * kWin;
        for (int e = threadIdx.x; e < kWin; e += kDepositThreads) slab[e] = W[e];
        __syncthreads();
    }
    // particles inside the outermost box: one LDS and one global add per workgroup
    atomicAdd(&cnt_sh, in0);
    __syncthreads();
    if (threadIdx.x == 0 && cnt_sh) atomicAdd(inside_count, (unsigned long long)cnt_sh);
}

__global__ void __launch_bounds__(kDepositThreads)
deposit_window_k(DepositArgs A, const double *__restrict__ x, const double *__restrict__ y,
                 const double *__restrict__ z, const double *__restrict__ m, int64_t np, int64_t per_block,
                 unsigned long long *__restrict__ inside_count)
{
    __shared__ unsigned long long W[kWin];
    __shared__ unsigned int cnt_sh;
    window_share(A, x, y, z, m, np, per_block, inside_count, W, cnt_sh);
}

// Node e of box b's window over the slabs g0 .. g1 - 1.
__device__ __forceinline__ unsigned long long window_sum(const DepositArgs &A, int g0, int g1, int e, int b)
{
    // four independent integer sums keep four slab loads in flight (any order gives the same sum)
    unsigned long long s0 = 0ULL, s1 = 0ULL, s2 = 0ULL, s3 = 0ULL;
    const size_t st = (size_t)A.nbox * kWin;
    const unsigned long long *src = A.scratch + (size_t)b * kWin + e;
    int g = g0;
    for (; g + 4 <= g1; g += 4) {
        s0 += src[(size_t)g * st];
        s1 += src[(size_t)(g + 1) * st];
        s2 += src[(size_t)(g + 2) * st];
        s3 += src[(size_t)(g + 3) * st];
    }
    for (; g < g1; ++g) s0 += src[(size_t)g * st];
    return (s0 + s1) + (s2 + s3);
}

// ... added to the grid
__device__ __forceinline__ void window_add(const DepositArgs &A, int e, int b, unsigned long long s)
{
    const int li = e % kWinX, lj = (e / kWinX) % kWinY, lk = e / (kWinX * kWinY);
    const int i = A.w0[b][0] + li, j = A.w0[b][1] + lj, k = A.w0[b][2] + lk;
    if (i >= A.n || j >= A.n || k >= A.n) return;
    if (s) A.q[b][id3(A.n, i, j, k)] += s;
}

__global__ void __launch_bounds__(256)
deposit_reduce_k(DepositArgs A, int nblocks)
{
    const int e = blockIdx.x * 256 + threadIdx.x, b = blockIdx.y;
    if (e < kWin) window_add(A, e, b, window_sum(A, 0, nblocks, e, b));
}

size_t deposit_scratch_bytes(int nbox) { return (size_t)kDepositMaxBlocks * nbox * kWin * sizeof(unsigned long long); }

void launch_deposit(const DepositArgs &a, const double *x, const double *y, const double *z, const double *m,
                    int64_t np, unsigned long long *inside_count, hipStream_t s)
{
    if (np <= 0) return;
    int64_t blocks = (np + kDepositThreads - 1) / kDepositThreads;
    if (blocks > kDepositMaxBlocks) blocks = kDepositMaxBlocks;
    const int64_t per_block = (np + blocks - 1) / blocks;
    hipLaunchKernelGGL(deposit_window_k, dim3((unsigned)blocks), dim3(kDepositThreads), 0, s, a, x, y, z, m, np,
                       per_block, inside_count);
    hipLaunchKernelGGL(deposit_reduce_k, dim3((kWin + 255) / 256, a.nbox), dim3(256), 0, s, a, (int)blocks);
}

// ------------------------------------------------------------ sorted deposit
//
// Where a disk is wider than the window above, most corners of large particle
// sets went to global 64-bit atomics, whose device-wide rate (about 17 G/s)
// bound the deposit.  The sorted form first orders the particles by the 32x32x8
// cell tile of the finest box that holds them, so that a workgroup takes
// particles of one tile and adds all their corners, on that box and on every
// coarser one, in LDS: in a box twice as large the tile is a block of half the
// cells per axis, and the blocks of all boxes together hold at most 11 645 nodes
// (93 KB).  Only the nodes a workgroup has touched go to the grids with global
// atomics, once per kSegment particles or more.  The weights, their rounding
// and the integer sums are those of the window form, so the grids are the same
// integers whatever the order.
//   0. deposit_start_k clears the grids and draws a sample of the particles, from
//      which it says whether the sorted form or the window form takes them;
//   1. deposit_first_k: LDS histogram over the tiles per workgroup, kept per
//      workgroup and added to the totals (or the window form's shares);
//   2. deposit_second_k: start of every tile, list of segments (or the sums of the
//      window form's slabs);
//   3. tile_scatter_k: particles as 32-byte records in tile order;
//   4. tile_deposit_k: segments from a queue.
// It is bound by its passes over the particles (24 + 32 + 32 + 32 B each) and by
// the eight rounded weights per particle and box.  Deposit calls (with clearing
// q and forming the right-hand side), window form -> sorted, of disks as wide as the
// finest box: 1e7 particles on 513^3 3944 -> 1111 us, in eleven 257^3 boxes 9.0 -> 2.0
// ms, 1e6 in three 257^3 boxes 985 -> 319 us, in four 129^3 boxes 526 -> 128 us.  1e7
// particles within a few cells of 129^3 are the window form's: sorted 323 us, now 156.

constexpr int kTileXY = 32, kTileZ = 8;
constexpr int kSortBlocks = kDepositMaxBlocks;   // the window form in these launches fills as many slabs
constexpr int kSegment = 4096;
constexpr int kWinAll = 11904;       // room for one tile's blocks on all boxes
constexpr int kWinOne = 33 * 33 * 9;

constexpr int blocks_of_all_boxes()
{
    int nodes = 0;
    for (int b = 0, xy = kTileXY, z = kTileZ; b < kMaxBox; ++b, xy = xy > 1 ? xy / 2 : 1, z = z > 1 ? z / 2 : 1)
        nodes += (xy + 1) * (xy + 1) * (z + 1);
    return nodes;
}
static_assert(blocks_of_all_boxes() == 11645 && blocks_of_all_boxes() <= kWinAll, "a tile's blocks fit");

struct TileGrid {
    int cxy, cz;      // cells per tile
    int sxy, sz;      // their logarithms
    int txy, tz;      // tiles per axis
    int per_box, nbin;
};

static TileGrid tile_grid(int n, int nbox)
{
    TileGrid t;
    const int m = n - 1;             // a power of two
    t.cxy = m < kTileXY ? m : kTileXY;
    t.cz = m < kTileZ ? m : kTileZ;
    t.sxy = __builtin_ctz((unsigned)t.cxy);
    t.sz = __builtin_ctz((unsigned)t.cz);
    t.txy = m / t.cxy;
    t.tz = m / t.cz;
    t.per_box = t.txy * t.txy * t.tz;
    t.nbin = t.per_box * nbox;
    return t;
}

// Tile of the finest box that holds the particle (the arithmetic of cic_cell), -1 outside all.
__device__ __forceinline__ int tile_of(const DepositArgs &A, const TileGrid &T, double px, double py, double pz, bool &in0)
{
#pragma clang fp contract(off)
    const double top = (double)(A.n - 1);
    int bin = -1;
    in0 = false;
    for (int b = A.nbox - 1; b >= 0; --b) {
        const BoxGeom &g = A.box[b];
        const double ux = (px - g.xmin) * g.inv_h, uy = (py - g.xmin) * g.inv_h, uz = (pz - g.xmin) * g.inv_h;
        const bool in = ux >= 0.0 && ux < top && uy >= 0.0 && uy < top && uz >= 0.0 && uz < top;
        if (b == 0) in0 = in;
        if (in && bin < 0)
            bin = b * T.per_box + (((int)uz >> T.sz) * T.txy + ((int)uy >> T.sxy)) * T.txy + ((int)ux >> T.sxy);
    }
    return bin;
}

// Which form is the faster one, from kSample particles, one of each of as many
// equal runs of the list.  Either form gives the same integers, so the choice is
// one of time alone.  What the forms cost, fitted to deposits of disks, spheres,
// uniform and compact sets of 2.5e5 to 1e7 particles on 129^3 to 513^3 (1 to 11
// boxes), in ps:
//   window  12 per particle and box, 340 per particle and box whose corners lie
//           outside the window (eight global atomics);
//   sorted  18.5 per particle, 10 per particle and box, 32000 per tile with
//           particles (its LDS window is cleared and scanned however few).
// So a set inside the window stays there (1e7 particles of a disk four cells
// wide, 129^3: 164 us against 339), as does one that is thin on the tiles
// (250 000 filling a 513^3 box: 842 against 1069).
constexpr int kStartThreads = 256, kSample = 2 * kStartThreads;
constexpr int kMaxTiles = 32768;

__device__ __forceinline__ void choose_form(const DepositArgs &A, const TileGrid &T, const double *__restrict__ x,
                                            const double *__restrict__ y, const double *__restrict__ z, int np,
                                            int *__restrict__ sorted)
{
    __shared__ unsigned seen[kMaxTiles / 32];   // a bit per tile
    __shared__ unsigned beyond, tiles;
    constexpr int NS = kSample / kStartThreads;
    double sx[NS], sy[NS], sz[NS];               // all in flight before the LDS is cleared
#pragma unroll
    for (int r = 0; r < NS; ++r) {
        const unsigned i = threadIdx.x + kStartThreads * r;
        // a place of its own in every run: lists have periods
        const float at = ((float)(i * 2654435769u) * 0x1p-32f) * ((float)np / kSample);
        const int p = min((int)((long long)i * np / kSample) + (int)at, np - 1);
        sx[r] = x[p];
        sy[r] = y[p];
        sz[r] = z[p];
    }
    for (int e = threadIdx.x; e < kMaxTiles / 32; e += kStartThreads) seen[e] = 0;
    if (threadIdx.x == 0) beyond = tiles = 0;
    __syncthreads();
    unsigned out = 0;
#pragma unroll
    for (int r = 0; r < NS; ++r) {
        const double px = sx[r], py = sy[r], pz = sz[r];
        bool in0;
        const int bin = tile_of(A, T, px, py, pz, in0);
        if (bin >= 0) atomicOr(&seen[bin >> 5], 1u << (bin & 31));
        for (int b = 0; b < A.nbox; ++b) {
            int ic[3];
            double w[3][2];
            if (!cic_cell(A.box[b], A.n, px, py, pz, ic, w)) continue;
            const int lx = ic[0] - A.w0[b][0], ly = ic[1] - A.w0[b][1], lz = ic[2] - A.w0[b][2];
            out += !(lx >= 0 && lx < kWinX - 1 && ly >= 0 && ly < kWinY - 1 && lz >= 0 && lz < kWinZ - 1);
        }
    }
    if (out) atomicAdd(&beyond, out);
    __syncthreads();
    unsigned hit = 0;
    for (int e = threadIdx.x; e < kMaxTiles / 32; e += kStartThreads) hit += __popc(seen[e]);
    if (hit) atomicAdd(&tiles, hit);
    __syncthreads();
    if (threadIdx.x >= 64) return;
    // t tiles hit evenly show t (1 - exp(-kSample / t)) of them: t from 64 values between the tiles seen and all
    const float d = (float)max(tiles, 1u);
    const float t = d * exp2f(log2f((float)T.nbin / d) * ((float)threadIdx.x / 63.0f));
    const unsigned long long below = __ballot(t * (1.0f - expf(-(float)kSample / t)) < d);
    if (threadIdx.x != min(__popcll(below), 63)) return;
    const float n = (float)np, nb = (float)A.nbox;
    const float window = 12.0f * nb * n + 340.0f * ((float)beyond / kSample) * n;
    const float sort = (18.5f + 10.0f * nb) * n + 32000.0f * t;
    *sorted = window > sort;
}

// Clears the totals, the count of particles (clear) and, where a sample is drawn
// (sorted), beside it the grids.
__global__ void __launch_bounds__(kStartThreads)
deposit_start_k(DepositArgs A, TileGrid T, const double *__restrict__ x, const double *__restrict__ y,
                const double *__restrict__ z, int np, int clear, unsigned *__restrict__ total,
                unsigned long long *__restrict__ inside_count, int *__restrict__ sorted)
{
    if (blockIdx.x == 0) {
        if (sorted) choose_form(A, T, x, y, z, np, sorted);
        return;
    }
    const size_t t = (blockIdx.x - 1) * (size_t)kStartThreads + threadIdx.x, st = (gridDim.x - 1) * (size_t)kStartThreads;
    for (size_t e = t; e < (size_t)T.nbin; e += st) total[e] = 0;
    if (!clear) return;
    if (t == 0) *inside_count = 0ULL;
    if (!sorted) return;
    // 16 bytes at a time on the small grids (deposit in one 257^3 box 145 -> 142 us, in
    // two 513^3 boxes 1456 -> 1540)
    const size_t N = (size_t)A.n * A.n * A.n;
    for (int b = 0; b < A.nbox; ++b) {
        if (A.n <= 257) {
            for (size_t e = 2 * t; e < N; e += 2 * st) {
                if (e + 1 < N) *reinterpret_cast<ulonglong2 *>(A.q[b] + e) = ulonglong2{0ULL, 0ULL};
                else A.q[b][e] = 0ULL;
            }
        } else {
            for (size_t e = t; e < N; e += st) A.q[b][e] = 0ULL;
        }
    }
}

template <int MAXBIN>
__device__ __forceinline__ void tile_count(const DepositArgs &A, const TileGrid &T, const double *__restrict__ x,
                                           const double *__restrict__ y, const double *__restrict__ z, int np,
                                           int per_block, unsigned *__restrict__ hist, unsigned *__restrict__ total,
                                           unsigned long long *__restrict__ inside_count, unsigned *H, unsigned &cnt_sh)
{
    for (int e = threadIdx.x; e < T.nbin; e += 1024) H[e] = 0;
    if (threadIdx.x == 0) cnt_sh = 0;
    __syncthreads();
    const int p0 = blockIdx.x * per_block, p1 = min(np, p0 + per_block);
    unsigned in_n = 0;
    for (int p = p0 + threadIdx.x; p < p1; p += 1024) {
        bool in0;
        const int bin = tile_of(A, T, x[p], y[p], z[p], in0);
        in_n += in0;
        if (bin >= 0) atomicAdd(&H[bin], 1u);
    }
    if (in_n) atomicAdd(&cnt_sh, in_n);
    __syncthreads();
    unsigned *row = hist + (size_t)blockIdx.x * T.nbin;
    for (int e = threadIdx.x; e < T.nbin; e += 1024) {
        const unsigned h = H[e];
        row[e] = h;
        if (h) atomicAdd(total + e, h);
    }
    if (threadIdx.x == 0 && cnt_sh) atomicAdd(inside_count, (unsigned long long)cnt_sh);
}

template <int MAXBIN>
__global__ void __launch_bounds__(1024)
deposit_first_k(DepositArgs A, TileGrid T, const double *__restrict__ x, const double *__restrict__ y,
                const double *__restrict__ z, const double *__restrict__ m, int np, int per_block,
                unsigned *__restrict__ hist, unsigned *__restrict__ total, unsigned long long *__restrict__ inside_count,
                const int *__restrict__ sorted)
{
    static_assert(MAXBIN <= 2 * kWin, "the histogram lies in the window's LDS");
    __shared__ unsigned long long W[kWin];
    __shared__ unsigned cnt_sh;
    if (!sorted || *sorted)
        tile_count<MAXBIN>(A, T, x, y, z, np, per_block, hist, total, inside_count, reinterpret_cast<unsigned *>(W), cnt_sh);
    else
        window_share(A, x, y, z, m, np, per_block, inside_count, W, cnt_sh);
}

// One workgroup: start[bin] = particles before the bin, next[bin] the same (the
// scatter's cursor); seg[] = {bin, first, end} of every segment of at most
// seg_len particles; queue[0] = number of segments, queue[1] = 0.
template <int MAXBIN>
__device__ __forceinline__ void tile_scan(int nbin, int seg_len, const unsigned *__restrict__ total,
                                          unsigned *__restrict__ next, int4 *__restrict__ seg, unsigned *__restrict__ queue)
{
    constexpr int PER = MAXBIN / 1024;               // bins per thread, in order
    __shared__ unsigned B[MAXBIN + 1024];            // one word of padding per thread's bins
    __shared__ unsigned sp[1024], ss[1024];
    for (int e = threadIdx.x; e < MAXBIN; e += 1024) B[e + e / PER] = e < nbin ? total[e] : 0u;
    __syncthreads();
    unsigned *mine = B + threadIdx.x * (PER + 1);
    unsigned np = 0, ns = 0;
    for (int k = 0; k < PER; ++k) {
        np += mine[k];
        ns += (mine[k] + seg_len - 1) / seg_len;
    }
    sp[threadIdx.x] = np;
    ss[threadIdx.x] = ns;
    __syncthreads();
    for (int d = 1; d < 1024; d <<= 1) {
        const unsigned a = (int)threadIdx.x >= d ? sp[threadIdx.x - d] : 0u;
        const unsigned c = (int)threadIdx.x >= d ? ss[threadIdx.x - d] : 0u;
        __syncthreads();
        sp[threadIdx.x] += a;
        ss[threadIdx.x] += c;
        __syncthreads();
    }
    unsigned p = sp[threadIdx.x] - np, s = ss[threadIdx.x] - ns;
    for (int k = 0; k < PER; ++k) {
        const unsigned c = mine[k];
        mine[k] = p;
        for (unsigned o = 0; o < c; o += seg_len)
            seg[s++] = make_int4(threadIdx.x * PER + k, (int)(p + o), (int)(p + min(c, o + seg_len)), 0);
        p += c;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < nbin; e += 1024) next[e] = B[e + e / PER];
    if (threadIdx.x == 1023) {
        queue[0] = ss[1023];
        queue[1] = 0;
    }
}

template <int MAXBIN>
__global__ void __launch_bounds__(1024)
deposit_second_k(DepositArgs A, int nbin, int seg_len, const unsigned *__restrict__ total, unsigned *__restrict__ next,
                 int4 *__restrict__ seg, unsigned *__restrict__ queue, const int *__restrict__ sorted)
{
    if (!sorted || *sorted) {
        if (blockIdx.x == 0 && blockIdx.y == 0) tile_scan<MAXBIN>(nbin, seg_len, total, next, seg, queue);
        return;
    }
    // 256 nodes a workgroup, each over four quarters of the slabs
    __shared__ unsigned long long part[1024];
    static_assert(kWin % 256 == 0 && kSortBlocks % 4 == 0, "whole workgroups and quarters");
    constexpr int Q = kSortBlocks / 4;
    const int e = blockIdx.x * 256 + (threadIdx.x & 255), b = blockIdx.y, q = threadIdx.x >> 8;
    part[threadIdx.x] = window_sum(A, q * Q, (q + 1) * Q, e, b);
    __syncthreads();
    if (q == 0)
        window_add(A, e, b, (part[threadIdx.x] + part[threadIdx.x + 256]) + (part[threadIdx.x + 512] + part[threadIdx.x + 768]));
}

template <int MAXBIN>
__global__ void __launch_bounds__(1024)
tile_scatter_k(DepositArgs A, TileGrid T, const double *__restrict__ x, const double *__restrict__ y,
               const double *__restrict__ z, const double *__restrict__ m, int np, int per_block,
               const unsigned *__restrict__ hist, unsigned *__restrict__ next, double4 *__restrict__ rec,
               const int *__restrict__ sorted)
{
    __shared__ unsigned H[MAXBIN];
    if (sorted && !*sorted) return;
    const unsigned *row = hist + (size_t)blockIdx.x * T.nbin;
    for (int e = threadIdx.x; e < T.nbin; e += 1024) {   // this workgroup's place in every tile it has particles of
        const unsigned h = row[e];
        H[e] = h ? atomicAdd(next + e, h) : 0u;
    }
    __syncthreads();
    const int p0 = blockIdx.x * per_block, p1 = min(np, p0 + per_block);
    for (int p = p0 + threadIdx.x; p < p1; p += 1024) {
        bool in0;
        const double px = x[p], py = y[p], pz = z[p];
        const int bin = tile_of(A, T, px, py, pz, in0);
        if (bin < 0) continue;
        rec[atomicAdd(&H[bin], 1u)] = double4{px, py, pz, m[p]};
    }
}

// Segments from the queue.  A thread adds the corners of its particles
// that share a cell in registers before they go to LDS (in the coarse boxes of a deep
// nesting a whole tile is a cell or two).
template <int WIN>
__global__ void __launch_bounds__(1024)
tile_deposit_k(DepositArgs A, TileGrid T, const double4 *__restrict__ rec, const int4 *__restrict__ seg,
               unsigned *__restrict__ queue, const int *__restrict__ sorted)
{
#pragma clang fp contract(off)
    __shared__ unsigned long long W[WIN];
    __shared__ int4 sg;
    __shared__ int more;
    if (sorted && !*sorted) return;
    const unsigned nseg = queue[0];
    for (;;) {
        if (threadIdx.x == 0) {
            const unsigned s = atomicAdd(queue + 1, 1u);
            more = s < nseg;
            if (more) sg = seg[s];
        }
        __syncthreads();
        if (!more) return;           // the queue only grows: every workgroup gets here
        const int bin = sg.x, first = sg.y, end = sg.z;
        const int bf = bin / T.per_box;
        int t = bin - bf * T.per_box;
        const int tx = t % T.txy;
        t /= T.txy;
        const int ty = t % T.txy, tz = t / T.txy;
        // the tile's cells on box bf, and on the coarser boxes: a box's middle half, (n - 1) / 4
        // cells from its face, is the next one
        const int off = (A.n - 1) / 4;
        const int flo[3] = {tx * T.cxy, ty * T.cxy, tz * T.cz};
        const int fhi[3] = {flo[0] + T.cxy - 1, flo[1] + T.cxy - 1, flo[2] + T.cz - 1};
        for (int e = threadIdx.x; e < WIN; e += 1024) W[e] = 0ULL;
        __syncthreads();
        for (int i0 = first + (int)threadIdx.x; i0 < end; i0 += 4096) {
            double4 r[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) r[k] = rec[min(i0 + 1024 * k, end - 1)];
            int lo[3] = {flo[0], flo[1], flo[2]}, hi[3] = {fhi[0], fhi[1], fhi[2]};
            int base = 0;
            for (int b = bf; b >= 0; --b) {
                const int nx = hi[0] - lo[0] + 2, ny = hi[1] - lo[1] + 2, nz = hi[2] - lo[2] + 2;
                const BoxGeom g = A.box[b];
                unsigned long long sum[8];
                int at = -1;         // LDS place of the cell whose corners are in sum
                auto flush = [&]() {
#pragma unroll
                    for (int c = 0; c < 8; ++c)
                        atomicAdd(&W[at + (c & 1) + nx * (((c >> 1) & 1) + ny * (c >> 2))], sum[c]);
                };
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    int ic[3];
                    double w[3][2];
                    if (i0 + 1024 * k >= end || !cic_cell(g, A.n, r[k].x, r[k].y, r[k].z, ic, w)) continue;
                    const int lx = ic[0] - lo[0], ly = ic[1] - lo[1], lz = ic[2] - lo[2];
                    const bool inwin = lx >= 0 && lx < nx - 1 && ly >= 0 && ly < ny - 1 && lz >= 0 && lz < nz - 1;
                    const int here = base + lx + nx * (ly + ny * lz);
                    if (inwin && here != at) {
                        if (at >= 0) flush();
                        at = here;
#pragma unroll
                        for (int c = 0; c < 8; ++c) sum[c] = 0ULL;
                    }
#pragma unroll
                    for (int c = 0; c < 8; ++c) {
                        const double wt = (w[0][c & 1] * w[1][(c >> 1) & 1]) * w[2][c >> 2];
                        const unsigned long long qv = (unsigned long long)__double2ll_rn((wt * r[k].w) * A.scale);
                        if (inwin) sum[c] += qv;
                        // a rounding of the two boxes' cell coordinates that differs at a tile's face
                        else atomicAdd(A.q[b] + id3(A.n, ic[0] + (c & 1), ic[1] + ((c >> 1) & 1), ic[2] + (c >> 2)), qv);
                    }
                }
                if (at >= 0) flush();
                base += nx * ny * nz;
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    lo[d] = off + (lo[d] >> 1);
                    hi[d] = off + (hi[d] >> 1);
                }
            }
        }
        __syncthreads();
        int lo[3] = {flo[0], flo[1], flo[2]}, hi[3] = {fhi[0], fhi[1], fhi[2]};
        int base = 0;
        for (int b = bf; b >= 0; --b) {
            const int nx = hi[0] - lo[0] + 2, ny = hi[1] - lo[1] + 2, nz = hi[2] - lo[2] + 2;
            for (int e = threadIdx.x; e < nx * ny * nz; e += 1024) {
                const unsigned long long v = W[base + e];
                if (v) atomicAdd(A.q[b] + id3(A.n, lo[0] + e % nx, lo[1] + e / nx % ny, lo[2] + e / nx / ny), v);
            }
            base += nx * ny * nz;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                lo[d] = off + (lo[d] >> 1);
                hi[d] = off + (hi[d] >> 1);
            }
        }
        __syncthreads();
    }
}

// Where the sorted form can be the faster one.  The window form alone stays at
// 65^3 and below, whose window holds most of a disk (1e7 particles: 163 us against
// 357, six nested boxes 823 against 912), for few particles (129^3, 1e5: 48
// against 59, 3e5: 68 against 63 us; 257^3, 1e5: 104 against 102), and where the
// tiles outgrow an LDS histogram (1025^3, or 513^3 in more than two boxes).
bool deposit_sorts(int n, int nbox, int64_t np)
{
    return n >= 129 && np >= 250000 && tile_grid(n, nbox).nbin <= kMaxTiles;
}

// Where a sample decides between the forms.  It costs up to 3 us (disks, one box:
// 1e6 particles on 257^3 126 -> 129 us; in three boxes the launches saved outweigh
// it, 3e6 particles 425 -> 419), and in the window form two launches that end at
// once: more than it can save below 1e6 particles on at most 257^3 (250 000 of the
// sets above: the sorted form takes at most 7 % longer there).
static int deposit_samples(int n, int np) { return n > 257 || np >= 1000000; }

constexpr int64_t kSortSlice = 1 << 26;   // particles sorted at a time

static size_t round256(size_t b) { return (b + 255) / 256 * 256; }

// A power of two, so that counts that creep up from call to call share a workspace.
int64_t deposit_sort_capacity(int64_t np)
{
    int64_t m = 1 << 18;
    while (m < np && m < kSortSlice) m *= 2;
    return m;
}

size_t deposit_sort_bytes(int n, int nbox, int64_t m)
{
    const TileGrid t = tile_grid(n, nbox);
    return round256((size_t)m * sizeof(double4)) + round256((size_t)kSortBlocks * t.nbin * 4) + 2 * round256((size_t)t.nbin * 4) +
           round256(((size_t)m / kSegment + t.nbin + 1) * sizeof(int4)) + 512;
}

template <int MAXBIN>
static void deposit_sorted(const DepositArgs &a, const TileGrid &t, const double *x, const double *y, const double *z,
                           const double *m, int np, bool clear, unsigned long long *inside_count, void *ws, hipStream_t s)
{
    char *w = (char *)ws;
    double4 *rec = (double4 *)w;
    w += round256((size_t)np * sizeof(double4));
    unsigned *hist = (unsigned *)w;
    w += round256((size_t)kSortBlocks * t.nbin * 4);
    unsigned *total = (unsigned *)w;
    w += round256((size_t)t.nbin * 4);
    unsigned *next = (unsigned *)w;
    w += round256((size_t)t.nbin * 4);
    int4 *seg = (int4 *)w;
    w += round256(((size_t)np / kSegment + t.nbin + 1) * sizeof(int4));
    unsigned *queue = (unsigned *)w;
    w += 256;
    int *sorted = deposit_samples(a.n, np) ? (int *)w : nullptr;   // null: the sorted form
    const int per_block = (np + kSortBlocks - 1) / kSortBlocks;
    // long enough that touched nodes are flushed rarely, short enough for some 1000 segments
    int seg_len = np / 1024;
    seg_len = (seg_len < kSegment ? kSegment : seg_len + kSegment - 1) / kSegment * kSegment;
    // the grids are cleared beside the sample, or, where none is drawn, by fills of their own
    const size_t N = (size_t)a.n * a.n * a.n;
    if (clear && !sorted)
        for (int b = 0; b < a.nbox; ++b) launch_fill<unsigned long long>(a.q[b], N, 0ULL, s);
    const size_t fill = ((clear && sorted ? N : (size_t)t.nbin) + kStartThreads - 1) / kStartThreads;
    hipLaunchKernelGGL(deposit_start_k, dim3(1 + (unsigned)(fill < 16384 ? fill : 16384)), dim3(kStartThreads), 0, s, a, t,
                       x, y, z, np, clear ? 1 : 0, total, inside_count, sorted);
    hipLaunchKernelGGL((deposit_first_k<MAXBIN>), dim3(kSortBlocks), dim3(1024), 0, s, a, t, x, y, z, m, np, per_block,
                       hist, total, inside_count, sorted);
    hipLaunchKernelGGL((deposit_second_k<MAXBIN>), sorted ? dim3(kWin / 256, a.nbox) : dim3(1), dim3(1024), 0, s, a, t.nbin,
                       seg_len, total, next, seg, queue, sorted);
    hipLaunchKernelGGL((tile_scatter_k<MAXBIN>), dim3(kSortBlocks), dim3(1024), 0, s, a, t, x, y, z, m, np, per_block,
                       hist, next, rec, sorted);
    if (a.nbox == 1)
        hipLaunchKernelGGL((tile_deposit_k<kWinOne>), dim3(512), dim3(1024), 0, s, a, t, rec, seg, queue, sorted);
    else
        hipLaunchKernelGGL((tile_deposit_k<kWinAll>), dim3(256), dim3(1024), 0, s, a, t, rec, seg, queue, sorted);
}

void launch_deposit_sorted(const DepositArgs &a, const double *x, const double *y, const double *z, const double *m,
                           int64_t np, unsigned long long *inside_count, void *ws, hipStream_t s)
{
    const TileGrid t = tile_grid(a.n, a.nbox);
    for (int64_t p = 0; p < np; p += kSortSlice) {
        const int c = (int)(np - p < kSortSlice ? np - p : kSortSlice);
        if (t.nbin <= 8192) deposit_sorted<8192>(a, t, x + p, y + p, z + p, m + p, c, p == 0, inside_count, ws, s);
        else deposit_sorted<kMaxTiles>(a, t, x + p, y + p, z + p, m + p, c, p == 0, inside_count, ws, s);
    }
}

// Batched single-box deposit: workgroup (g, p) takes a contiguous share of
// problem p's particles, with the same LDS window, scratch slabs and integer
// adds as above; problem p's grid starts at q + p n^3.
__global__ void __launch_bounds__(kDepositThreads)
deposit_batch_k(int n, BoxGeom g, int wx, int wy, int wz, const BatchProblem *__restrict__ prob,
                unsigned long long *__restrict__ qall, unsigned long long *__restrict__ scratch,
                unsigned long long *__restrict__ inside)
{
#pragma clang fp contract(off)
    __shared__ unsigned long long W[kWin];
    __shared__ unsigned int cnt_sh;
    const int pb = blockIdx.y;
    const BatchProblem P = prob[pb];
    const int64_t per_block = (P.np + kBatchDepositBlocks - 1) / kBatchDepositBlocks;
    const int64_t p0 = (int64_t)blockIdx.x * per_block;
    const int64_t p1 = min((int64_t)P.np, p0 + per_block);
    unsigned long long *q = qall + (size_t)pb * n * n * n;
    if (threadIdx.x == 0) cnt_sh = 0;
    for (int e = threadIdx.x; e < kWin; e += kDepositThreads) W[e] = 0ULL;
    __syncthreads();
    unsigned int in0 = 0;
    for (int64_t p = p0 + threadIdx.x; p < p1; p += kDepositThreads) {
        int ic[3];
        double w[3][2];
        if (!cic_cell(g, n, P.x[p], P.y[p], P.z[p], ic, w)) continue;
        ++in0;
        const double pm = P.m[p];
        const int lx = ic[0] - wx, ly = ic[1] - wy, lz = ic[2] - wz;
        const bool inwin = lx >= 0 && lx < kWinX - 1 && ly >= 0 && ly < kWinY - 1 && lz >= 0 && lz < kWinZ - 1;
        for (int c = 0; c < 2; ++c)
            for (int bb = 0; bb < 2; ++bb)
                for (int a = 0; a < 2; ++a) {
                    const double wt = (w[0][a] * w[1][bb]) * w[2][c];
                    const unsigned long long qv = (unsigned long long)__double2ll_rn((wt * pm) * P.scale);
                    if (inwin) atomicAdd(&W[(lx + a) + kWinX * ((ly + bb) + kWinY * (lz + c))], qv);
                    else atomicAdd(q + id3(n, ic[0] + a, ic[1] + bb, ic[2] + c), qv);
                }
    }
    __syncthreads();
    unsigned long long *slab = scratch + ((size_t)pb * kBatchDepositBlocks + blockIdx.x) * kWin;
    for (int e = threadIdx.x; e < kWin; e += kDepositThreads) slab[e] = W[e];
    atomicAdd(&cnt_sh, in0);
    __syncthreads();
    if (threadIdx.x == 0 && cnt_sh) atomicAdd(inside + pb, (unsigned long long)cnt_sh);
}

__global__ void __launch_bounds__(256)
deposit_batch_reduce_k(int n, int wx, int wy, int wz, unsigned long long *__restrict__ qall,
                       const unsigned long long *__restrict__ scratch)
{
    const int e = blockIdx.x * 256 + threadIdx.x;
    const int pb = blockIdx.y;
    if (e >= kWin) return;
    const int li = e % kWinX, lj = (e / kWinX) % kWinY, lk = e / (kWinX * kWinY);
    const int i = wx + li, j = wy + lj, k = wz + lk;
    if (i >= n || j >= n || k >= n) return;
    unsigned long long s = 0ULL;
    for (int g = 0; g < kBatchDepositBlocks; ++g) s += scratch[((size_t)pb * kBatchDepositBlocks + g) * kWin + e];
    if (s) qall[(size_t)pb * n * n * n + id3(n, i, j, k)] += s;
}

size_t deposit_batch_scratch_bytes(int nb)
{
    return (size_t)nb * kBatchDepositBlocks * kWin * sizeof(unsigned long long);
}

void launch_deposit_batch(int n, double L, const BatchProblem *prob, long long maxnp, unsigned long long *q,
                          unsigned long long *scratch, unsigned long long *inside, int nb, hipStream_t s)
{
    (void)maxnp;
    BoxGeom g;
    g.L = L;
    g.xmin = -0.5 * L;
    g.inv_h = (double)(n - 1) / L;
    g.h = L / (double)(n - 1);
    const int win[3] = {kWinX, kWinY, kWinZ};
    int w0[3];
    for (int d = 0; d < 3; ++d) {
        const int o = (n - 1) / 2 - win[d] / 2;
        w0[d] = o < 0 ? 0 : o;
    }
    hipLaunchKernelGGL(deposit_batch_k, dim3(kBatchDepositBlocks, nb), dim3(kDepositThreads), 0, s, n, g, w0[0], w0[1],
                       w0[2], prob, q, scratch, inside);
    hipLaunchKernelGGL(deposit_batch_reduce_k, dim3((kWin + 255) / 256, nb), dim3(256), 0, s, n, w0[0], w0[1], w0[2], q,
                       scratch);
}

__global__ void rhs_from_q_k(size_t count, double inv_h3, double four_pi_G, int shift, const long long *__restrict__ q,
                             double *__restrict__ f)
{
    for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < count; t += (size_t)gridDim.x * blockDim.x) {
        const double rho = ldexp((double)q[t], -shift) * inv_h3;
        f[t] = four_pi_G * rho;
    }
}

void launch_rhs_from_q(int n, double h, double four_pi_G, int shift, const long long *q, double *f, hipStream_t s)
{
    const size_t count = (size_t)n * n * n;
    size_t blocks = (count + 255) / 256;
    if (blocks > 16384) blocks = 16384;
    hipLaunchKernelGGL(rhs_from_q_k, dim3((unsigned)blocks), dim3(256), 0, s, count, 1.0 / (h * h * h), four_pi_G,
                       shift, q, f);
}

// Problem blockIdx.y; q and f may alias (each element is read before it is written).
__global__ void rhs_batch_k(size_t count, double inv_h3, double four_pi_G, const BatchProblem *__restrict__ prob,
                            const long long *q, double *f)
{
    const int shift = prob[blockIdx.y].shift;
    q += blockIdx.y * count;
    f += blockIdx.y * count;
    for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < count; t += (size_t)gridDim.x * blockDim.x) {
        const double rho = ldexp((double)q[t], -shift) * inv_h3;
        f[t] = four_pi_G * rho;
    }
}

void launch_rhs_batch(int n, double h, double four_pi_G, const BatchProblem *prob, const long long *q, double *f, int nb,
                      hipStream_t s)
{
    const size_t count = (size_t)n * n * n;
    size_t blocks = (count + 255) / 256;
    if (blocks > 2048) blocks = 2048;
    hipLaunchKernelGGL(rhs_batch_k, dim3((unsigned)blocks, nb), dim3(256), 0, s, count, 1.0 / (h * h * h), four_pi_G,
                       prob, q, f);
}

// ------------------------------------------------------------------- gather
//
// The gather arithmetic is written out with contraction off, so that every
// kernel that inlines it (forces, curves, batched curves) rounds the same way.

// -d Phi / d x_d at node (i,j,k): central difference inside, one-sided second
// order on the faces.
__device__ __forceinline__ double node_accel(const double *__restrict__ P, int n, double inv2h, int i, int j, int k, int d)
{
#pragma clang fp contract(off)
    const size_t st = d == 0 ? 1 : (d == 1 ? (size_t)n : (size_t)n * n);
    const int c = d == 0 ? i : (d == 1 ? j : k);
    const size_t p = id3(n, i, j, k);
    double g;
    if (c > 0 && c < n - 1) g = P[p + st] - P[p - st];
    else if (c == 0) g = -3.0 * P[p] + 4.0 * P[p + st] - P[p + 2 * st];
    else g = 3.0 * P[p] - 4.0 * P[p - st] + P[p - 2 * st];
    return -g * inv2h;
}

// nu(y) with y = g / a0 (g > 0, a0 > 0): Eq. 2's function for nun == 1, else the n-family.
__device__ __forceinline__ double nu_of_g(double g, double a0, double nun)
{
#pragma clang fp contract(off)
    return nun == 1.0 ? 0.5 + 0.5 * sqrt(1.0 + 4.0 * a0 / g) : nu_family(g / a0, nun);
}

// Point-mass force (QUMOND: nu(g_N/a0) g_N) for points outside every box.
__device__ __forceinline__ void monopole_accel(double GM, double a0, int mond, double nun, double px, double py,
                                               double pz, double acc[3])
{
#pragma clang fp contract(off)
    const double r = sqrt(px * px + py * py + pz * pz);
    double g = 0.0;
    if (r > 0.0) {
        const double gN = GM / (r * r);
        g = (mond && a0 > 0.0 && gN > 0.0) ? nu_of_g(gN, a0, nun) * gN : gN;
        g /= r;
    }
    acc[0] = -g * px;
    acc[1] = -g * py;
    acc[2] = -g * pz;
}

__device__ __forceinline__ bool in_box(const BoxGeom &G, int n, double px, double py, double pz)
{
    const double top = (double)(n - 1);
    const double ux = (px - G.xmin) * G.inv_h, uy = (py - G.xmin) * G.inv_h, uz = (pz - G.xmin) * G.inv_h;
    return ux >= 0.0 && ux < top && uy >= 0.0 && uy < top && uz >= 0.0 && uz < top;
}

// Cloud-in-cell interpolation of the nodal accelerations of box G.  Cells whose
// corners all have central differences (all but the outermost layer) take the
// 32 nodes they need as 16 loads of x-pairs, all in flight at once; per node and
// direction the general form below made 48 loads in branches, one waiting for
// the other.  Same operations in the same order.  Bound by the cache lines a
// point touches: 4e6 points in two 257^3 boxes 677 -> 262 us, 1e7 on 513^3 1628
// -> 638 us; the curve of 60 radii and 16 azimuths 7.7 -> 5.0 us.
// On 5^3, with 8 such cells of 64, a wavefront goes through both forms: there the general one alone.
__device__ __forceinline__ void box_accel(const BoxGeom &G, int n, const double *__restrict__ P, double px, double py,
                                          double pz, double acc[3])
{
#pragma clang fp contract(off)
    typedef double pair_t __attribute__((ext_vector_type(2), aligned(8)));
    const double u[3] = {(px - G.xmin) * G.inv_h, (py - G.xmin) * G.inv_h, (pz - G.xmin) * G.inv_h};
    int ic[3];
    double w[3][2];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double fl = floor(u[d]);
        ic[d] = (int)fl;
        const double fr = u[d] - fl;
        w[d][0] = 1.0 - fr;
        w[d][1] = fr;
    }
    const double inv2h = 0.5 * G.inv_h;
    acc[0] = acc[1] = acc[2] = 0.0;
    if (n > 5 && min(min(ic[0], ic[1]), ic[2]) >= 1 && max(max(ic[0], ic[1]), ic[2]) <= n - 3) {
        const size_t sy = (size_t)n, sz = (size_t)n * n;
        const double *c0 = P + id3(n, ic[0], ic[1], ic[2]);
        auto at = [&](const double *p) { return *reinterpret_cast<const pair_t *>(p); };
        pair_t xl[2][2], xr[2][2], ym[2], yp[2], zm[2], zp[2];   // [z][y] (i - 1, i), (i + 1, i + 2); (i, i + 1) beside
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                xl[c][b] = at(c0 + c * sz + b * sy - 1);
                xr[c][b] = at(c0 + c * sz + b * sy + 1);
            }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            ym[t] = at(c0 + t * sz - sy);
            yp[t] = at(c0 + t * sz + 2 * sy);
            zm[t] = at(c0 + t * sy - sz);
            zp[t] = at(c0 + t * sy + 2 * sz);
        }
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int a = 0; a < 2; ++a) {
                    const double wt = (w[0][a] * w[1][b]) * w[2][c];
                    auto mid = [&](int cc, int bb) { return a ? xr[cc][bb].x : xl[cc][bb].y; };   // node i + a
                    const double gx = a ? xr[c][b].y - xl[c][b].y : xr[c][b].x - xl[c][b].x;
                    const double gy = b ? (a ? yp[c].y : yp[c].x) - mid(c, 0) : mid(c, 1) - (a ? ym[c].y : ym[c].x);
                    const double gz = c ? (a ? zp[b].y : zp[b].x) - mid(0, b) : mid(1, b) - (a ? zm[b].y : zm[b].x);
                    acc[0] += wt * (-gx * inv2h);
                    acc[1] += wt * (-gy * inv2h);
                    acc[2] += wt * (-gz * inv2h);
                }
        return;
    }
    for (int c = 0; c < 2; ++c)
        for (int b = 0; b < 2; ++b)
            for (int a = 0; a < 2; ++a) {
                const double wt = (w[0][a] * w[1][b]) * w[2][c];
                for (int d = 0; d < 3; ++d) acc[d] += wt * node_accel(P, n, inv2h, ic[0] + a, ic[1] + b, ic[2] + c, d);
            }
}

// Eq. 3, the algebraic MOND relation: g = nu(|g_N| / a0) g_N at the point.
__device__ __forceinline__ void algebraic_mond(double a0, double nun, double acc[3])
{
#pragma clang fp contract(off)
    const double g = sqrt(acc[0] * acc[0] + acc[1] * acc[1] + acc[2] * acc[2]);
    if (g > 0.0 && a0 > 0.0) {
        const double k = nu_of_g(g, a0, nun);
        acc[0] *= k;
        acc[1] *= k;
        acc[2] *= k;
    }
}

__device__ int gather_point(const GatherArgs &A, double px, double py, double pz, double acc[3])
{
#pragma clang fp contract(off)
    const double R = sqrt(px * px + py * py), az = fabs(pz);
    int sel = -1;
    for (int b = A.nbox - 1; b >= 0; --b)
        if (R < A.frac * A.box[b].L && az < A.frac * A.box[b].L) { sel = b; break; }
    if (sel < 0) {
        for (int b = 0; b < A.nbox; ++b)
            if (in_box(A.box[b], A.n, px, py, pz)) { sel = b; break; }
    }
    if (sel < 0) monopole_accel(A.GM, A.a0, A.mond, A.nun, px, py, pz, acc);
    else box_accel(A.box[sel], A.n, A.phi[sel], px, py, pz, acc);
    if (A.alg) algebraic_mond(A.a0, A.nun, acc);
    return sel < 0 ? 255 : sel;
}

__global__ void __launch_bounds__(256)
gather_k(GatherArgs A, const double *__restrict__ x, const double *__restrict__ y, const double *__restrict__ z,
         int64_t np, double *__restrict__ ax, double *__restrict__ ay, double *__restrict__ az, uint8_t *__restrict__ used)
{
    const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (p >= np) return;
    double acc[3];
    const int sel = gather_point(A, x[p], y[p], z[p], acc);
    ax[p] = acc[0];
    ay[p] = acc[1];
    az[p] = acc[2];
    if (used) used[p] = (uint8_t)sel;
}

void launch_gather(const GatherArgs &a, const double *x, const double *y, const double *z, int64_t np, double *ax,
                   double *ay, double *az, uint8_t *box_used, hipStream_t s)
{
    if (np <= 0) return;
    const int64_t blocks = (np + 255) / 256;
    hipLaunchKernelGGL(gather_k, dim3((unsigned)blocks), dim3(256), 0, s, a, x, y, z, np, ax, ay, az, box_used);
}

// Sum over the workgroup in the order of a tree over 256 threads.  A workgroup
// of one wavefront (64 threads, for at most 64 samples) skips the levels that
// would add zeros and needs no barriers.
__device__ __forceinline__ double tree_sum(double s, double *sh)
{
    if (blockDim.x == 64) {
#pragma unroll
        for (int w = 32; w > 0; w >>= 1) s += __shfl_down(s, w);
        return s;
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    return sh[0];
}

// Eq. 4 on the midplane: one workgroup per radius, azimuths phi_k = 2 pi k / naz,
// v_c^2 = -(x a_x + y a_y) averaged in a fixed order.
__global__ void __launch_bounds__(256)
rotation_curve_k(GatherArgs A, const double *__restrict__ R, int naz, double *__restrict__ vc2)
{
#pragma clang fp contract(off)
    __shared__ double sh[256];
    const double r = R[blockIdx.x];
    double s = 0.0;
    for (int k = threadIdx.x; k < naz; k += blockDim.x) {
        const double phi = 2.0 * M_PI * (double)k / (double)naz;
        const double px = r * cos(phi), py = r * sin(phi);
        double acc[3];
        gather_point(A, px, py, 0.0, acc);
        s += -(px * acc[0] + py * acc[1]);
    }
    s = tree_sum(s, sh);
    if (threadIdx.x == 0) vc2[blockIdx.x] = s / (double)naz;
}

void launch_rotation_curve(const GatherArgs &a, const double *R, int nR, int naz, double *vc2, hipStream_t s)
{
    if (nR <= 0) return;
    hipLaunchKernelGGL(rotation_curve_k, dim3(nR), dim3(naz <= 64 ? 64 : 256), 0, s, a, R, naz, vc2);
}

// Eq. 5 for stars with a sech^2(z / z0) vertical profile at every radius:
// rho / d_z rho = -z0 / (2 tanh(z / z0)), so sigma_z^2 = -a_z z0 / (2 tanh(z / z0)).
// One workgroup per radius; samples k < naz at (R cos phi_k, R sin phi_k, +z),
// k >= naz at the same azimuths and -z, averaged in a fixed order.
__global__ void __launch_bounds__(256)
sigma_z_k(GatherArgs A, const double *__restrict__ R, int naz, double z, double z0, double *__restrict__ sig2)
{
#pragma clang fp contract(off)
    __shared__ double sh[256];
    const double r = R[blockIdx.x];
    const double c = z0 / (2.0 * tanh(z / z0));
    double s = 0.0;
    for (int k = threadIdx.x; k < 2 * naz; k += blockDim.x) {
        const bool up = k < naz;
        const int ka = up ? k : k - naz;
        const double phi = 2.0 * M_PI * (double)ka / (double)naz;
        const double px = r * cos(phi), py = r * sin(phi);
        double acc[3];
        gather_point(A, px, py, up ? z : -z, acc);
        s += up ? -acc[2] * c : acc[2] * c;  // tanh is odd
    }
    s = tree_sum(s, sh);
    if (threadIdx.x == 0) sig2[blockIdx.x] = s / (double)(2 * naz);
}

void launch_sigma_z(const GatherArgs &a, const double *R, int nR, int naz, double z, double z0, double *sig2,
                    hipStream_t s)
{
    if (nR <= 0) return;
    hipLaunchKernelGGL(sigma_z_k, dim3(nR), dim3(2 * naz <= 64 ? 64 : 256), 0, s, a, R, naz, z, z0, sig2);
}

// Batched single-box curves: workgroup (r, p), same sampling and order as rotation_curve_k.
__global__ void __launch_bounds__(256)
rotation_curve_batch_k(int n, BoxGeom G, double frac, double Gc, double a0, int mond, double nun,
                       const BatchProblem *__restrict__ prob, const double *__restrict__ phi, const double *__restrict__ R,
                       int nR, int naz, double *__restrict__ vc2)
{
#pragma clang fp contract(off)
    __shared__ double sh[256];
    const int pb = blockIdx.y;
    const double *P = phi + (size_t)pb * n * n * n;
    const double GM = Gc * prob[pb].mass;
    const double r = R[blockIdx.x];
    double s = 0.0;
    for (int k = threadIdx.x; k < naz; k += blockDim.x) {
        const double ph = 2.0 * M_PI * (double)k / (double)naz;
        const double px = r * cos(ph), py = r * sin(ph);
        double acc[3];
        // the box-choice rule of gather_point with one box
        const double Rp = sqrt(px * px + py * py);
        if ((Rp < frac * G.L && 0.0 < frac * G.L) || in_box(G, n, px, py, 0.0)) box_accel(G, n, P, px, py, 0.0, acc);
        else monopole_accel(GM, a0, mond, nun, px, py, 0.0, acc);
        s += -(px * acc[0] + py * acc[1]);
    }
    s = tree_sum(s, sh);
    if (threadIdx.x == 0) vc2[(size_t)pb * nR + blockIdx.x] = s / (double)naz;
}

void launch_rotation_curve_batch(int n, double L, double frac, double G, double a0, int mond,
                                 const BatchProblem *prob, const double *phi, const double *R, int nR, int naz,
                                 double *vc2, int nb, hipStream_t s, double nun)
{
    if (nR <= 0 || nb <= 0) return;
    BoxGeom g;
    g.L = L;
    g.xmin = -0.5 * L;
    g.inv_h = (double)(n - 1) / L;
    g.h = L / (double)(n - 1);
    hipLaunchKernelGGL(rotation_curve_batch_k, dim3(nR, nb), dim3(naz <= 64 ? 64 : 256), 0, s, n, g, frac, G, a0, mond, nun, prob, phi,
                       R, nR, naz, vc2);
}

}  // namespace qm
