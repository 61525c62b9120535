// Two red-black Gauss-Seidel sweeps in one pass over u and f (Sec. 2: the
// smoother of the multigrid solves of Eq. 1 and Eq. 2), with the four
// half-sweeps of a z-march skewed one plane apart.
//
// A thread owns one x-pair of nodes (one red, one black: i + j + k even and
// odd) of the tile plus a four-node ring and marches along z.  Step s updates
// the red node of plane s (first sweep), the black one of plane s - 1 (first
// sweep), the red one of plane s - 2 (second sweep) and the black one of plane
// s - 3 (second sweep).  A node's z neighbours and one of its x neighbours
// belong to its own thread and stay in registers, those of this step among
// them; only the other x neighbour and the two y neighbours come from LDS, on
// the same plane, where the stage before left them in the step before.  So
// LDS holds two half-planes (one colour) per stage, indexed by the thread: all
// accesses of a wavefront are consecutive, the twelve reads of a step are
// independent, and one barrier per plane separates the steps.  Of a pair, all
// four stages of a step update the same node.  Every node update sees exactly
// the values it sees in two sequential sweeps.  In x and y each stage covers
// one ring fewer than the one before (the tile plus three, two, one and zero
// nodes), recomputing the neighbours' ring nodes from the same inputs, so the
// tile's values equal the sequential sweeps' bit for bit.  A plane of u and of
// f is requested two steps before use.
//
// A workgroup marches planes K0 .. K1 - 1 of its column: the whole column, or a
// chunk of it on grids whose columns alone leave CUs idle (257^3: 64 columns of
// 64x16 for 256 CUs).  A chunk needs u four planes and the stages three, two
// and one plane beyond its ends, which it recomputes as it does the ring: the
// march starts at step K0 - 3 and ends with step K1 + 2, and what the stages
// write further out is read by no value that is kept.
//
// Bound: 513^3 by HBM (two sweeps move 24 B per node once: 595 us FP64 = 5.4
// TB/s), smaller grids by the step's issue and latency (about 0.7 us on 64x16
// columns), FP32 by both.  The form before this one skewed the stages two planes
// apart and read all six neighbours from ten LDS planes of both colours, at a
// stride of two values: 1.4 us per step, 726 us at 513^3.  Loads that are not
// masked, LDS writes without a branch and, away from the column's ends, steps
// without range checks came after: FP32 513^3 425 -> 406 us, 257^3 51 -> 45 (with
// the correction 77 -> 68), FP64 257^3 90 -> 88 (110 -> 107).  Requesting planes
// four steps ahead gained nothing.  FP64 pairs, before -> now (with
// the correction): 513^3 726 -> 595 (862 -> 697) us; 257^3, there two single
// sweeps, 203 -> 88 (235 -> 107) us in 64-plane chunks; 129^3 45 -> 17 (59 -> 23)
// us in 8-plane chunks; 65^3, there 8^3 bricks, 18 -> 9 (26 -> 11) us.  64x16
// columns waste least on the ring (1.7 nodes per node of the tile; 1.9 at 32x16,
// 2.5 at 32x8) and win from 129^3 up; the small ones fill the chip at 65^3.
#include "common.h"

namespace qm {

namespace {

// ZERO: the iterate is zero (uin is not read).  PROLONG: the coarse-grid
// correction u += P uc (uc on the grid of nc = (n + 1) / 2 points) is added to
// every interior node as its plane enters the march, with the trilinear
// expression of the prolong-add kernel evaluated in the same order (along x,
// then y, then z) on coarse planes staged in LDS, so the result is that of a
// prolong-add launch followed by the two sweeps, bit for bit.
template <typename T, int TX, int TY, int NT, bool ZERO, bool PROLONG>
__global__ void __launch_bounds__(NT)
rbgs2_skew_k(const T *__restrict__ uin, T *__restrict__ uout, const T *__restrict__ f, int n, T h2,
             const T *__restrict__ uc, int nc, int kchunk, int nchunk)
{
#pragma clang fp contract(off)
    typedef T pair_t __attribute__((ext_vector_type(2), aligned(sizeof(T))));
    constexpr int RG = 4;                                  // ring of the region a workgroup owns
    constexpr int HP = TX / 2 + RG, PY = TY + 2 * RG, NP = HP * PY;   // its x-pairs and rows
    static_assert(TX % 2 == 0 && TY % 2 == 0 && NP <= NT, "one pair of nodes per thread");
    constexpr int PAD = HP + 1, ROW = NT + 2 * PAD;        // reads of the outermost threads stay inside
    // coarse rows of the region (tile origins are odd): TY / 2 + 5; a coarse
    // plane is staged interpolated along x on the region's fine columns, the
    // even and the odd of a pair apart
    constexpr int CPY = TY / 2 + 5, XPL = 2 * HP * CPY, NXL = (XPL + NT - 1) / NT;
    __shared__ T half[4][2][ROW];   // [black, red 1, black 1, red 2][plane parity]
    __shared__ T cpl[PROLONG ? 3 : 1][PROLONG ? XPL : 1];   // coarse plane c, along x, in slot c % 3
    const T sixth = T(1) / T(6);
    const int tid = threadIdx.x;
    const unsigned tl = xcd_tile(blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z),
                                 gridDim.x * gridDim.y * gridDim.z);
    const int bx = tl % gridDim.x, by = (tl / gridDim.x) % gridDim.y, bz = tl / (gridDim.x * gridDim.y);
    const int pb = bz / nchunk, ch = bz - pb * nchunk;
    // kchunk is even and at least 4, so every march starts with an odd step
    const int K0 = max(1, ch * kchunk), K1 = min(n - 1, (ch + 1) * kchunk);
    const int s0 = max(1, K0 - 3), umax = min(n - 1, K1 + 3), fmax = min(n - 2, K1 + 2);
    const int i0 = 1 + bx * TX, j0 = 1 + by * TY;
    const size_t nn = (size_t)n * n;
    if (!ZERO) uin += (size_t)pb * nn * n;
    uout += (size_t)pb * nn * n;
    f += (size_t)pb * nn * n;
    if (PROLONG) uc += (size_t)pb * nc * nc * nc;

    // This thread's pair: nodes (il, jp), (il + 1, jp).  Bit 2w + e of ok says
    // that node e is an interior node on the tile plus a ring of width w.
    const int q = tid % HP, br = tid / HP;
    const int il = i0 - RG + 2 * q, jp = j0 - RG + br;
    unsigned ok = 0;
    if (tid < NP && jp >= 1 && jp <= n - 2) {
#pragma unroll
        for (int w = 0; w < 4; ++w)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int a = 2 * q + e, i = il + e;
                if (a >= RG - w && a <= RG + TX - 1 + w && br >= RG - w && br <= RG + TY - 1 + w && i >= 1 && i <= n - 2)
                    ok |= 1u << (2 * w + e);
            }
    }
    const int me = PAD + tid;                  // LDS place of the pair
    // u of the pair on a plane: one 16-byte load, its place clamped into the plane
    // (the node before a row's first is the row before's last; a row outside the
    // grid and threads beyond the region read the tile's corner pair, since lanes
    // of all workgroups meeting on one cache line would queue on it).  Nothing is
    // masked: what is no node of the grid, or lies on one of its edges, enters no
    // update that is kept.
    const int idle = i0 + n * j0;
    auto bytes = [](int p) { return (unsigned)p * (unsigned)sizeof(T); };
    const unsigned uoff = bytes(tid < NP && jp >= 0 && jp < n ? min(max(il + n * jp, 0), n * n - 2) : idle);
    auto at = [](const T *g, unsigned off) {
        return *reinterpret_cast<const pair_t *>(reinterpret_cast<const char *>(g) + off);
    };
    auto fetch = [&](const T *g, pair_t &v) {
        if (!ZERO) v = at(g, uoff);
    };
    // f of the pair (in range: both columns lie in the grid when either is
    // interior on the widest ring)
    const unsigned foff = bytes((ok >> 6) != 0 ? il + n * jp : idle);
    auto f_pair = [&](const T *g) { return at(g, foff); };

    // The correction's coarse data: per staged entry r of this thread (pair t %
    // HP, parity and coarse row from t / HP), the two coarse nodes its
    // x-interpolation weighs (xo, or -1 where the column is not interior or the
    // row is outside the grid: a lane with nothing to load reads the first of
    // the region's coarse nodes); odd columns of the grid are interpolated.
    const int cj0 = (j0 - RG) >> 1;
    int xo[NXL];
    bool xodd[NXL];
    const int cidle = max((i0 - RG) >> 1, 0) + nc * max(cj0, 0);
    if constexpr (PROLONG) {
#pragma unroll
        for (int r = 0; r < NXL; ++r) {
            const int t = tid + r * NT;
            const int e = (t / HP) & 1, i = i0 - RG + 2 * (t % HP) + e, J = cj0 + t / (2 * HP);
            xo[r] = (t < XPL && i >= 1 && i <= n - 2 && J >= 0 && J < nc) ? (i >> 1) + nc * J : -1;
            xodd[r] = i & 1;
        }
    }
    T cv0[NXL], cv1[NXL];
    auto fetch_c = [&](int c) {   // the coarse nodes of plane c (clamped into the grid) into cv0, cv1
        if constexpr (PROLONG) {
            const char *C = reinterpret_cast<const char *>(uc + (size_t)min(c, nc - 1) * nc * nc);
#pragma unroll
            for (int r = 0; r < NXL; ++r) {
                const unsigned o = bytes(xo[r] >= 0 ? xo[r] : cidle);
                cv0[r] = *reinterpret_cast<const T *>(C + o);
                cv1[r] = *reinterpret_cast<const T *>(C + (xodd[r] && xo[r] >= 0 ? o + (unsigned)sizeof(T) : o));
            }
        }
    };
    // ... interpolated along x into its LDS slot (prolong_at's x step: weights 1, 0 at even columns, 1/2, 1/2 at odd)
    auto store_c = [&](int c) {
        if constexpr (PROLONG) {
            if (c > nc - 1) return;
#pragma unroll
            for (int r = 0; r < NXL; ++r) {
                const int t = tid + r * NT;
                if (t >= XPL) continue;
                const T wia = xodd[r] ? T(0.5) : T(1), wib = xodd[r] ? T(0.5) : T(0);
                cpl[c % 3][t] = xo[r] >= 0 ? wia * cv0[r] + wib * cv1[r] : T(0);
            }
        }
    };
    // the correction at node e of the pair on plane k (1 <= k <= n - 2):
    // prolong_at's y and z steps on the staged planes
    const int dj = jp & 1, crow = q + 2 * HP * max((jp >> 1) - cj0, 0);
    const bool jin = tid < NP && jp >= 1 && jp <= n - 2;
    const bool cin0 = jin && il >= 1 && il <= n - 2, cin1 = jin && il + 1 >= 1 && il + 1 <= n - 2;
    auto corr = [&](int e, int k) {
        const T wja = dj ? T(0.5) : T(1), wjb = dj ? T(0.5) : T(0);
        const T wka = (k & 1) ? T(0.5) : T(1), wkb = (k & 1) ? T(0.5) : T(0);
        const T *Xa = cpl[(k >> 1) % 3], *Xb = cpl[((k + 1) >> 1) % 3];
        const int o = crow + e * HP, oj = o + dj * 2 * HP;
        const T xa = Xa[o], xb = Xa[oj], xc = Xb[o], xd = Xb[oj];
        return wka * (wja * xa + wjb * xb) + wkb * (wja * xc + wjb * xd);
    };
    // The pair's red and black value as plane k enters (er: the red node).  With
    // the correction only the black one takes it: a red node's own value is
    // replaced by the first sweep's red update before any update reads it, and
    // red nodes of the outer ring are not read at all.
    auto enter = [&](int k, const pair_t &v, int er, bool inside, T &r, T &b) {
        const T x0 = ZERO ? T(0) : v.x, x1 = ZERO ? T(0) : v.y;
        r = er ? x1 : x0;
        b = er ? x0 : x1;
        if (PROLONG && (inside || (k >= 1 && k <= n - 2)) && (er ? cin0 : cin1)) b += corr(er ^ 1, k);
    };

    // Own values by plane.  Before step s: bz[0], bz[1] = black of planes s - 1, s
    // as they entered; ra = red of plane s; r1 = red of planes s - 1, s - 2 after
    // the first sweep; b1 = black of planes s - 2, s - 3; r2 = red of planes
    // s - 3, s - 4 after the second.  hr, hb: h^2 f of the red node of planes
    // s - 1, s - 2 and of the black node of planes s - 1 .. s - 3.
    T bzm, bzc, ra, r1a, r1b, b1a = T(0), b1b = T(0), r2a = T(0), r2b = T(0);
    T hr1 = T(0), hr2 = T(0), hb1 = T(0), hb2 = T(0), hb3 = T(0);
    // warm-up: planes s0 - 1 and s0 enter (with the correction: coarse planes
    // e, e + 1, e + 2 first, e = (s0 - 1) / 2); planes s0 + 1, s0 + 2, the f pairs
    // of planes s0, s0 + 1 and coarse plane e + 3 in flight
    int er = (il + jp + s0) & 1;         // the red node of the pair on plane s0
    {
        pair_t w0 = {T(0), T(0)}, w1 = {T(0), T(0)};
        fetch(uin + (size_t)(s0 - 1) * nn, w0);
        fetch(uin + (size_t)s0 * nn, w1);
        if constexpr (PROLONG) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                fetch_c((s0 - 1) / 2 + c);
                store_c((s0 - 1) / 2 + c);
            }
            __syncthreads();
        }
        enter(s0 - 1, w0, er ^ 1, false, r1a, bzm);
        enter(s0, w1, er, false, ra, bzc);
        r1b = T(0);
    }
    fetch_c((s0 - 1) / 2 + 3);
    pair_t vA = {T(0), T(0)}, vB = {T(0), T(0)};
    // in the order of the loop's requests, which its waits count; pu and pf: the
    // next planes of u and f, clamped into the march's (what the last steps fetch
    // beyond them is never used)
    auto plane = [&](const T *g, int k) { return g + (size_t)k * nn; };
    fetch(plane(uin, min(s0 + 1, umax)), vA);
    pair_t pA = f_pair(plane(f, min(s0, fmax)));
    __builtin_amdgcn_sched_barrier(0);
    fetch(plane(uin, min(s0 + 2, umax)), vB);
    pair_t pB = f_pair(plane(f, min(s0 + 1, fmax)));
    __builtin_amdgcn_sched_barrier(0);
    const T *pu = plane(uin, min(s0 + 3, umax)), *pf = plane(f, min(s0 + 2, fmax));
    half[0][s0 & 1][me] = bzc;
    __syncthreads();

    const int smax = K1 + 2;   // the last black update of the second sweep is plane K1 - 1
    T *const dst0 = uout + (ptrdiff_t)n * jp + il;
    // even: s is even (the loop's second step of a pair); with the correction,
    // an even step s stores coarse plane (s + 4) / 2, first read by fine plane
    // s + 3, which enters in step s + 2, and requests plane (s + 6) / 2
    // inside: all four updates' planes are interior and plane s - 3 is one of the chunk's
    auto step = [&](int s, pair_t &vX, pair_t &pX, const bool even, const bool inside) {
        const int p = even ? 0 : 1;      // parity of plane s, s - 2
        const int xn = me + (er ? 1 : -1);
        // the three lateral neighbours of the four updates
        const T ax = half[0][p][xn], ad = half[0][p][me - HP], au = half[0][p][me + HP];
        const T bx1 = half[1][p ^ 1][xn], bd = half[1][p ^ 1][me - HP], bu = half[1][p ^ 1][me + HP];
        const T cx = half[2][p][xn], cd = half[2][p][me - HP], cu = half[2][p][me + HP];
        const T dx = half[3][p ^ 1][xn], dd = half[3][p ^ 1][me - HP], du = half[3][p ^ 1][me + HP];
        const unsigned m = ok >> er;
        // plane s + 1 enters
        T rn, bn;
        enter(s + 1, vX, er ^ 1, inside, rn, bn);
        const T hr0 = h2 * (er ? pX.y : pX.x), hb0 = h2 * (er ? pX.x : pX.y);
        if (PROLONG && even) {   // into the slot of coarse plane s / 2 - 1, last read in step s - 2
            store_c((s + 4) / 2);
            fetch_c((s + 6) / 2);
        }
        fetch(pu, vX);
        pX = f_pair(pf);
        pu += s + 3 < umax ? nn : 0;
        pf += s + 2 < fmax ? nn : 0;
        // sums in the order of the single sweep (x, y, z neighbours; the two of x commute)
        const T r1n = ((inside || s <= n - 2) && (m & 64)) ? (bzc + ax + ad + au + bzm + bn - hr0) * sixth : ra;
        const T b1n = ((inside || (s - 1 >= 1 && s - 1 <= n - 2)) && (m & 16))
                          ? (r1a + bx1 + bd + bu + r1b + r1n - hb1) * sixth : bzm;
        const T r2n = ((inside || (s - 2 >= 1 && s - 2 <= n - 2)) && (m & 4))
                          ? (b1a + cx + cd + cu + b1b + b1n - hr2) * sixth : r1b;
        const T b2n = (r2a + dx + dd + du + r2b + r2n - hb3) * sixth;
        half[0][p ^ 1][me] = bn;
        half[1][p][me] = r1n;
        half[2][p ^ 1][me] = b1n;
        half[3][p][me] = r2n;
        // plane s - 3 is final: its black node is node er of the pair
        const int k = s - 3;
        if ((inside || (k >= K0 && k < K1)) && (ok & 3)) {
            T *dst = dst0 + (size_t)k * nn;
            if ((ok & 3) == 3) {
                pair_t o;
                o.x = er ? r2a : b2n;
                o.y = er ? b2n : r2a;
                *reinterpret_cast<pair_t *>(dst) = o;
            } else {                     // one node of the pair is on the far face
                dst[ok & 2 ? 1 : 0] = (er != 0) == ((ok & 2) != 0) ? b2n : r2a;
            }
        }
        bzm = bzc;
        bzc = bn;
        ra = rn;
        r1b = r1a;
        r1a = r1n;
        b1b = b1a;
        b1a = b1n;
        r2b = r2a;
        r2a = r2n;
        hr2 = hr1;
        hr1 = hr0;
        hb3 = hb2;
        hb2 = hb1;
        hb1 = hb0;
        er ^= 1;
        __syncthreads();
    };
    // whole pairs of steps: no branch inside a loop; those with every plane inside
    // check none (not with the correction: a second copy of its step spills, 813 us
    // at 513^3 in FP64 against 697)
    const int sa = PROLONG ? smax : max(K0 + 3, s0 + 2), sb = min(n - 3, smax - 1);
    int s = s0;
    for (; s < sa && s + 1 <= smax; s += 2) {
        step(s, vA, pA, false, false);
        step(s + 1, vB, pB, true, false);
    }
    if constexpr (!PROLONG) {
        for (; s <= sb; s += 2) {
            step(s, vA, pA, false, true);
            step(s + 1, vB, pB, true, true);
        }
        for (; s + 1 <= smax; s += 2) {
            step(s, vA, pA, false, false);
            step(s + 1, vB, pB, true, false);
        }
    }
    if (s <= smax) step(s, vA, pA, false, false);
}

}  // namespace

template <typename T, int TX, int TY, int NT>
static void skew_launch(int n, double h, const T *f, const T *uin, T *uout, hipStream_t s, int nb, const T *uc, int kchunk)
{
    const int m = n - 2;
    // chunk c holds planes max(1, c kchunk) .. (c + 1) kchunk - 1 of 1 .. n - 2
    const int kc = kchunk <= 0 || kchunk >= n - 1 ? n - 1 : (kchunk < 4 ? 4 : kchunk + (kchunk & 1));
    const int nchunk = (n - 1 + kc - 1) / kc;
    const dim3 grid((m + TX - 1) / TX, (m + TY - 1) / TY, nb * nchunk);
    const int nc = (n + 1) / 2;
    if (uc)
        hipLaunchKernelGGL((rbgs2_skew_k<T, TX, TY, NT, false, true>), grid, dim3(NT), 0, s, uin, uout, f, n, T(h * h),
                           uc, nc, kc, nchunk);
    else if (uin)
        hipLaunchKernelGGL((rbgs2_skew_k<T, TX, TY, NT, false, false>), grid, dim3(NT), 0, s, uin, uout, f, n, T(h * h),
                           uc, nc, kc, nchunk);
    else
        hipLaunchKernelGGL((rbgs2_skew_k<T, TX, TY, NT, true, false>), grid, dim3(NT), 0, s, uin, uout, f, n, T(h * h),
                           uc, nc, kc, nchunk);
}

template <typename T>
void launch_rbgs2_skew(int n, double h, const T *f, const T *uin, T *uout, hipStream_t s, int nb, const T *uc, int tile,
                       int kchunk)
{
    if (tile == 1) skew_launch<T, 32, 8, 320>(n, h, f, uin, uout, s, nb, uc, kchunk);
    else if (tile == 2) skew_launch<T, 32, 16, 512>(n, h, f, uin, uout, s, nb, uc, kchunk);
    else skew_launch<T, 64, 16, 896>(n, h, f, uin, uout, s, nb, uc, kchunk);
}

template void launch_rbgs2_skew<double>(int, double, const double *, const double *, double *, hipStream_t, int,
                                        const double *, int, int);
template void launch_rbgs2_skew<float>(int, double, const float *, const float *, float *, hipStream_t, int,
                                       const float *, int, int);

}  // namespace qm
