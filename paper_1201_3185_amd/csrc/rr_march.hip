// Residual and full-weighting restriction of one level marching in z (the
// coarse right-hand side of the multigrid solves of Eq. 1 and Eq. 2).
//
// A workgroup owns CX x CY coarse columns and a chunk of kc coarse planes.  A
// thread owns the 2 x 2 fine nodes of one coarse column (or of the ring around
// the workgroup's) and marches along z.  Step p forms their residuals on plane
// p: the z neighbours and half of the x and y ones are the thread's own, in
// registers, the others come from an LDS plane of u written the step before.
// In the same step the thread adds the nine residuals of plane p - 1 around its
// coarse node, four of them its own and five from an LDS plane, to a running
// sum: an even plane is the centre of its coarse plane, an odd one ends the sum
// of the plane below and begins that of the plane above with the same nine
// products.  Both LDS planes are double, so one barrier separates the steps,
// and hold the four classes of nodes apart, so all accesses of a wavefront are
// consecutive.  Each residual and each coarse sum is the expression of
// residual_restrict_k in its order, so the results are the same bits.  A plane
// of u is requested three steps before use, one of f two.
//
// Bound: 257^3 and up by HBM (16 B read per fine node, FP64; 513^3 503 us = 4.5
// TB/s, 257^3 62 us), smaller grids by the step's latency (0.55 us a plane), so
// they take small tiles and short chunks.  The kernel before this one formed the
// residuals of two planes between barriers from four LDS planes of u, with all
// nine residuals of every coarse sum from LDS three planes deep, two barriers a
// plane pair and masked loads.  Residual restriction before -> now, FP64 (FP32):
// 129^3 19.5 -> 12.4 (15.6 -> 9.9), 257^3 85.5 -> 61.8 (49.0 -> 31.5), 513^3
// 520 -> 503 (294 -> 291) us.
//
// Chunks: without one given (kc 0), a column is cut until every CU has a workgroup
// (FP32: two).  More of them only form the planes between chunks twice: 32 x 8
// columns at 257^3, whole, 128, 64, 32 and 16 planes: 182, 181, 100, 62 and 63 us (FP32 122,
// 120, 65, 38 and 31), at 513^3 511, 578, 686, 669 and 664 (308, 306, 334, 365 and
// 370).  So from 513^3 up, where whole columns fill the chip, a shorter chunk is
// not taken either (16 x 8 columns in 4, 8 and 16 planes 879, 743 and 685 us, whole 570).
// Of many grids at once the chip's last, part-filled turn counts too: nine of 257^3 in
// FP32 373 us in chunks of 64 planes, 358 in chunks of 16, which the tuning of a batch
// finds.
//
// No value is masked: what is loaded outside the grid (clamped addresses) or
// formed on the ring only enters residuals that no interior coarse node reads.
#include <algorithm>

#include "common.h"

namespace qm {

namespace {

template <typename T, int CX, int CY, int NT>
__global__ void __launch_bounds__(NT)
rr_march_k(int nf, T ih2, const T *__restrict__ f, const T *__restrict__ u, T *__restrict__ fc, T *__restrict__ uc0,
           T *__restrict__ uc1, int tx, int ty, int tzc, int kc, int zu)
{
#pragma clang fp contract(off)
    typedef T pair_t __attribute__((ext_vector_type(2), aligned(sizeof(T))));   // global: any alignment
    constexpr int HP = CX + 2, NP = HP * (CY + 2);   // coarse columns of the region
    static_assert(NP <= NT, "one coarse column per thread");
    constexpr int PAD = HP + 1, ROW = NT + 2 * PAD;   // reads of the outermost threads stay inside
    // [plane parity][class of node: 2 (row parity) + column parity; residuals: less 1]
    __shared__ T Us[2][4][ROW], Rs[2][3][ROW];
    const int nc = (nf + 1) / 2;
    int bid = (int)xcd_tile(blockIdx.x, gridDim.x);
    const int bx = bid % tx;
    bid /= tx;
    const int by = bid % ty;
    bid /= ty;
    const int bz = bid % tzc;
    const int pb = bid / tzc;
    const size_t Nf = (size_t)nf * nf * nf, Nc = (size_t)nc * nc * nc, sz = (size_t)nf * nf;
    f += pb * Nf;
    u += pb * Nf;
    fc += pb * Nc;
    uc0 += pb * Nc;
    if (uc1) uc1 += pb * Nc;
    const int tid = threadIdx.x;
    const int I0 = 1 + bx * CX, J0 = 1 + by * CY;   // first coarse column
    const int Kb = 1 + bz * kc, Ke = min(Kb + kc - 1, nc - 2);

    // This thread's nodes: columns 2I, 2I + 1 of rows 2J, 2J + 1, a row loaded as
    // one pair.  Rows are clamped into the grid, and a pair into its plane: the
    // node after a row's last is the next row's first, the plane's last pair
    // holds the corner's value in the wrong place.  Neither enters an interior
    // residual, nor do the threads beyond the region's.
    const int q = tid % HP, br = tid / HP, me = PAD + tid;
    const int I = I0 - 1 + q, J = J0 - 1 + br;
    auto place = [&](int j) { return (unsigned)min(2 * I + nf * min(j, nf - 1), nf * nf - 2) * (unsigned)sizeof(T); };
    const unsigned off0 = place(2 * J), off1 = place(2 * J + 1);
    struct quad {
        pair_t a, b;   // rows 2J and 2J + 1
    };
    auto load = [&](const T *plane) {
        const char *c = reinterpret_cast<const char *>(plane);
        return quad{*reinterpret_cast<const pair_t *>(c + off0), *reinterpret_cast<const pair_t *>(c + off1)};
    };
    auto hold = [](quad &v) { asm volatile("" : "+v"(v.a.x), "+v"(v.a.y), "+v"(v.b.x), "+v"(v.b.y)); };
    auto put_u = [&](T (*U)[ROW], quad v) {
        U[0][me] = v.a.x;
        U[1][me] = v.a.y;
        U[2][me] = v.b.x;
        U[3][me] = v.b.y;
    };

    // the owner of a coarse column next to the low faces also zeroes the boundary
    // column beyond it
    const bool c_thread = q >= 1 && q <= CX && br >= 1 && br <= CY && I < nc && J < nc;
    const bool c_inner = c_thread && I <= nc - 2 && J <= nc - 2;
    auto zero_at = [&](int Ix, int Jx, int K) {
        const size_t C = id3(nc, Ix, Jx, K);
        uc0[C] = T(0);
        if (uc1) uc1[C] = T(0);
        fc[C] = T(0);
    };
    const int Z0 = bz == 0 ? 0 : Kb, Z1 = bz == tzc - 1 ? nc - 1 : Ke;
    for (int K = Z0; c_thread && K <= Z1; ++K) {
        if (!c_inner || K == 0 || K == nc - 1) zero_at(I, J, K);
        if (I == 1) zero_at(0, J, K);
        if (J == 1) zero_at(I, 0, K);
        if (I == 1 && J == 1) zero_at(0, 0, K);
    }

    const int p0 = 2 * Kb - 1;   // first residual plane (odd)
    const T *u0 = u + (size_t)(p0 - 1) * sz, *f0 = f + (size_t)p0 * sz;
    quad wm = load(u0), w0 = load(u0 + sz), wp = load(u0 + 2 * sz);
    // u(p + 2) and f(p) of the odd and the even steps, in the order of the steps
    quad ua = load(u0 + 3 * sz), fa = load(f0);
    __builtin_amdgcn_sched_barrier(0);
    quad ub = load(u0 + 4 * sz), fb = load(f0 + sz);
    __builtin_amdgcn_sched_barrier(0);
    const T *pu = u + (size_t)min(p0 + 4, nf - 1) * sz, *pf = f0 + 2 * sz;   // the next planes, clamped into the grid
    quad r = {};   // the thread's residuals of plane p - 1
    put_u(Us[1], w0);
    T acc = T(0);
    __syncthreads();

    // One step on plane p of parity B: residuals from Us[B], u(p + 1) to
    // Us[1 - B], residuals to r and Rs[B]; the nine residuals of plane p - 1 in r9.
    auto step = [&](const int B, quad &un, quad &fn, T (&r9)[9]) {
        const T xm0 = Us[B][1][me - 1], xp0 = Us[B][0][me + 1], xm1 = Us[B][3][me - 1], xp1 = Us[B][2][me + 1];
        const T ym0 = Us[B][2][me - HP], ym1 = Us[B][3][me - HP], yp0 = Us[B][0][me + HP], yp1 = Us[B][1][me + HP];
        r9[0] = Rs[1 - B][2][me - HP - 1];
        r9[1] = Rs[1 - B][1][me - HP];
        r9[2] = Rs[1 - B][2][me - HP];
        r9[3] = Rs[1 - B][0][me - 1];
        r9[4] = r.a.x;
        r9[5] = r.a.y;
        r9[6] = Rs[1 - B][2][me - 1];
        r9[7] = r.b.x;
        r9[8] = r.b.y;
        put_u(Us[1 - B], wp);
        quad fv = fn;
        hold(fv);
        r.a.x = fv.a.x - (xm0 + w0.a.y + ym0 + w0.b.x + wm.a.x + wp.a.x - T(6) * w0.a.x) * ih2;
        r.a.y = fv.a.y - (w0.a.x + xp0 + ym1 + w0.b.y + wm.a.y + wp.a.y - T(6) * w0.a.y) * ih2;
        r.b.x = fv.b.x - (xm1 + w0.b.y + w0.a.x + yp0 + wm.b.x + wp.b.x - T(6) * w0.b.x) * ih2;
        r.b.y = fv.b.y - (w0.b.x + xp1 + w0.a.y + yp1 + wm.b.y + wp.b.y - T(6) * w0.b.y) * ih2;
        Rs[B][0][me] = r.a.y;
        Rs[B][1][me] = r.b.x;
        Rs[B][2][me] = r.b.y;
        wm = w0;
        w0 = wp;
        wp = un;
        hold(wp);
    };
    // The loads of two steps on, after all uses of the registers they fill (the
    // held copies): otherwise they go elsewhere and are copied, and waited for,
    // at the end of the loop.
    auto refill = [&](int p, quad &un, quad &fn) {
        __builtin_amdgcn_sched_barrier(0);
        un = load(pu);
        fn = load(pf);
        pu += p + 4 < nf - 1 ? sz : 0;
        pf += p + 2 < nf - 1 ? sz : 0;
    };
    // the weights are powers of two: their products are exact, and an FMA is the
    // multiplication and the addition
    const T w[3] = {T(0.25), T(0.5), T(0.25)};
    for (int K = Kb; K <= Ke + 1; ++K) {
        T r9[9];
        step(1, ua, fa, r9);   // r9: plane 2K - 2, the centre of K - 1
#pragma unroll
        for (int e = 0; e < 9; ++e) acc = fma(w[e % 3] * w[e / 3] * T(0.5), r9[e], acc);
        refill(2 * K - 1, ua, fa);
        __syncthreads();
        step(0, ub, fb, r9);   // r9: plane 2K - 1, above K - 1 and below K
        T next = T(0);
#pragma unroll
        for (int e = 0; e < 9; ++e) {
            const T c = w[e % 3] * w[e / 3] * T(0.25);
            acc = fma(c, r9[e], acc);
            next = fma(c, r9[e], next);
        }
        if (c_inner && K > Kb) {
            const size_t C = id3(nc, I, J, K - 1);
            fc[C] = acc;
            if (zu) uc0[C] = T(0);
        }
        acc = next;
        refill(2 * K, ub, fb);
        __syncthreads();
    }
}

template <typename T, int CX, int CY, int NT>
void launch_tiles(int nf, double h, const T *f, const T *u, T *fc, T *uc0, T *uc1, int kc, hipStream_t s, int nb, int zu)
{
    const int nc = (nf + 1) / 2;
    const int tx = (nc - 1 + CX - 1) / CX, ty = (nc - 1 + CY - 1) / CY;
    // the shortest chunk that leaves no more workgroups than one (FP32: two) for each of the 256 CUs
    const long long want = sizeof(T) == 8 ? 256 : 512, tiles = (long long)tx * ty * nb;
    const int fill = (int)((nc - 2) / ((want + tiles - 1) / tiles)) + 1;
    if (kc <= 0 || nf >= 513) kc = std::max(kc, fill);
    kc = std::min(kc, nc - 2);
    const int tzc = (nc - 2 + kc - 1) / kc;
    hipLaunchKernelGGL((rr_march_k<T, CX, CY, NT>), dim3((unsigned)((size_t)tx * ty * tzc * nb)), dim3(NT), 0, s, nf,
                       T(1.0 / (h * h)), f, u, fc, uc0, uc1, tx, ty, tzc, kc, zu);
}

}   // namespace

template <typename T>
void launch_rr_march(int nf, double h, const T *f, const T *u, T *fc, T *uc0, T *uc1, int wide, int kc, hipStream_t s,
                     int nb, int zu)
{
    if (wide)
        launch_tiles<T, 32, 8, 384>(nf, h, f, u, fc, uc0, uc1, kc, s, nb, zu);
    else
        launch_tiles<T, 16, 8, 192>(nf, h, f, u, fc, uc0, uc1, kc, s, nb, zu);
}

template void launch_rr_march<double>(int, double, const double *, const double *, double *, double *, double *, int,
                                      int, hipStream_t, int, int);
template void launch_rr_march<float>(int, double, const float *, const float *, float *, float *, float *, int, int,
                                     hipStream_t, int, int);

}   // namespace qm
