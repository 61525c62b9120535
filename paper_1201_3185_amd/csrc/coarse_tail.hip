// The coarse tail of the multigrid solves (Sec. 2 of Angus et al.): every level
// with at most 17 points per side inside one workgroup, so that a V-cycle or a
// whole FMG over these levels is one launch.  Level l has 2^l + 1 points; the
// 3^3 level is solved exactly, in FP64.
//
// A thread owns the 2 x 2 x 2 nodes (2q + e) of a block q of a level and keeps
// their u and f in registers for the whole launch, on every level at once.  A
// node's colour and its place among the eight follow from e alone, so every
// register index is a constant and a phase has no index arithmetic: in LDS each
// level has one array per e, [q], and a thread's accesses are one address and
// constant offsets.  A node reads three neighbours from LDS and has three of its
// own.  Rows of an array hold the blocks alone, the far face of x follows them:
// with the face in the rows, at a stride of nine values, every access took twice
// the LDS cycles in conflicts.  Block q of a level is also node q of the level below it, which the same
// thread restricts to (eight of the 27 residuals are its own) and prolongs from.
// 17^3 has 512 owners, 9^3 64 and 5^3 eight: the levels below 17^3 belong to the
// first wavefront, which works through them in order and without barriers, while
// the others wait at one.  The far faces (2q + 2 of the last block) are boundary
// nodes only and live in LDS alone.
//
// No value is masked on its way in: what is read beyond a low face only enters
// boundary nodes, which keep their values.
//
// Bound by the latency and the instruction issue of its dependent phases.  With a
// pair of nodes per thread (1024 threads, four LDS reads a node at 17^3, places
// and colours worked out in every phase) a V-cycle from 17^3 took 12.1 us, now
// 9.1 (from 9^3 5.0 -> 4.4; from 5^3, eight lanes' work, 2.0 -> 2.2).
#include "common.h"

namespace qm {

namespace {

constexpr int kTailTop = 4;

template <int LV>
struct Lv {
    static constexpr int n = (1 << LV) + 1, NQ = 1 << (LV - 1), Q = NQ + 1;   // blocks of a row; with the far face
    static constexpr int S = Q * Q * Q, SR = NQ * NQ * NQ;                    // a class of nodes of u, of residuals
    static constexpr int OWN = SR;
};

// LDS, in values: the residuals of levels 4, 3, 2 (classes 1 to 7), their u, the
// restricted right-hand sides of levels 3 and 2, u of the 3^3 level
constexpr int kPad = 128;   // reads beyond the low faces of the first array
template <int LV> __host__ __device__ constexpr int at_r()
{
    return LV == 4 ? kPad : at_r<LV == 4 ? 4 : LV + 1>() + 7 * Lv<LV == 4 ? 4 : LV + 1>::SR + 8 * Lv<LV == 4 ? 4 : LV + 1>::S;
}
template <int LV> __host__ __device__ constexpr int at_u() { return at_r<LV>() + 7 * Lv<LV>::SR; }
template <int LV> __host__ __device__ constexpr int at_f()
{
    return LV == 3 ? at_u<2>() + 8 * Lv<2>::S : at_u<2>() + 8 * Lv<2>::S + Lv<4>::SR;
}
constexpr int kAtU1 = at_f<2>() + Lv<3>::SR, kTailLds = kAtU1 + 27;

template <typename T, int LV>
struct Own {
    T u[8], f[8];           // node e = ex + 2 ey + 4 ez of the block
    int at, ar;             // the block's place in the arrays of u and of residuals
    int xp;                 // ... of u of the next block of the row, or the far face
    int qx, qy, qz;
    bool act, low[3];       // low[d]: the block lies on the low face of direction d

    __device__ void init()
    {
        constexpr int NQ = Lv<LV>::NQ, Q = Lv<LV>::Q;
        const int t = threadIdx.x % Lv<LV>::OWN;
        act = (int)threadIdx.x < Lv<LV>::OWN;
        qx = t % NQ;
        qy = t / NQ % NQ;
        qz = t / (NQ * NQ);
        at = (qz * Q + qy) * NQ + qx;
        xp = qx < NQ - 1 ? at + 1 : (NQ * Q + qz) * Q + qy;
        ar = t;
        low[0] = qx == 0;
        low[1] = qy == 0;
        low[2] = qz == 0;
    }
    // The indices count as new from here: addresses of every phase kept across the cycles would spill.
    __device__ void fresh() { asm volatile("" : "+v"(at), "+v"(xp), "+v"(ar), "+v"(qx), "+v"(qy), "+v"(qz)); }
    __device__ bool interior(int e) const
    {
        return !((!(e & 1) && low[0]) || (!(e & 2) && low[1]) || (!(e & 4) && low[2]));
    }
};

template <typename T, int TOP>
struct Tail {
    T *mem;
    double L;
    T h2, ih2;               // h^2 and 1 / h^2 of the top level
    int npre, npost;
    Own<T, 4> o4;
    Own<T, 3> o3;
    Own<T, 2> o2;
    T f1;

    template <int LV> __device__ Own<T, LV> &own()
    {
        if constexpr (LV == 4) return o4;
        else if constexpr (LV == 3) return o3;
        else return o2;
    }
    // Levels up to 9^3 belong to the first wavefront, whose LDS operations complete in order.
    template <int LV> __device__ static void sync()
    {
        if constexpr (LV >= 4) {
            __syncthreads();
        } else {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    }
    template <int LV> __device__ static bool mine() { return LV >= 4 || threadIdx.x < 64; }

    // sum of the six neighbours of node e, in grid order (the two of x commute)
    template <int LV> __device__ T neighbours(const Own<T, LV> &o, int e)
    {
#pragma clang fp contract(off)
        constexpr int NQ = Lv<LV>::NQ, P = Lv<LV>::Q * NQ, S = Lv<LV>::S;
        const T *U = mem + at_u<LV>() + o.at, *X = mem + at_u<LV>() + o.xp;
        const T xo = e & 1 ? X[(e ^ 1) * S] : U[(e ^ 1) * S - 1];
        const T yo = U[(e ^ 2) * S + (e & 2 ? NQ : -NQ)], yi = o.u[e ^ 2];
        const T zo = U[(e ^ 4) * S + (e & 4 ? P : -P)], zi = o.u[e ^ 4];
        return o.u[e ^ 1] + xo + (e & 2 ? yi : yo) + (e & 2 ? yo : yi) + (e & 4 ? zi : zo) + (e & 4 ? zo : zi);
    }
    static __device__ constexpr int colour(int e) { return (e ^ e >> 1 ^ e >> 2) & 1; }
    // the block's values to LDS: those of one colour, or all (2)
    template <int LV, int C> __device__ void put_u(const Own<T, LV> &o)
    {
        if (LV > 2 || o.act) {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (C == 2 || colour(e) == C) mem[at_u<LV>() + o.at + e * Lv<LV>::S] = o.u[e];
        }
    }
    template <int LV, int C> __device__ void pass()
    {
#pragma clang fp contract(off)
        Own<T, LV> &o = own<LV>();
        const T hh = h2 * T(1 << 2 * (TOP - LV)), sixth = T(1) / T(6);
        T v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (colour(e) == C) v[e] = (neighbours<LV>(o, e) - hh * o.f[e]) * sixth;
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (colour(e) == C) o.u[e] = o.interior(e) ? v[e] : o.u[e];
        put_u<LV, C>(o);
        sync<LV>();
    }
    template <int LV> __device__ void sweeps(int ns)
    {
        for (int s = 0; s < ns; ++s) {
            pass<LV, 0>();
            pass<LV, 1>();
        }
    }
    // Full weighting of v (a value per node of level LV) at the block's coarse
    // node, in the order of the restriction kernel; meaningful inside the low faces.
    template <int LV> __device__ T weighted(const T (&v)[8])
    {
#pragma clang fp contract(off)
        constexpr int NQ = Lv<LV>::NQ, SR = Lv<LV>::SR;
        Own<T, LV> &o = own<LV>();
        T *R = mem + at_r<LV>() + o.ar - SR;
        if (LV > 2 || o.act) {
#pragma unroll
            for (int e = 1; e < 8; ++e) R[e * SR] = v[e];
        }
        sync<LV>();
        const T w[3] = {T(0.25), T(0.5), T(0.25)};
        T acc = T(0);
#pragma unroll
        for (int c = -1; c <= 1; ++c)
#pragma unroll
            for (int b = -1; b <= 1; ++b)
#pragma unroll
                for (int a = -1; a <= 1; ++a) {
                    const int e = (a & 1) + 2 * (b & 1) + 4 * (c & 1);
                    const int d = (a < 0 ? 1 : 0) + (b < 0 ? NQ : 0) + (c < 0 ? NQ * NQ : 0);
                    const T x = d == 0 ? v[e] : R[e * SR - d];
                    acc += (w[a + 1] * w[b + 1] * w[c + 1]) * x;
                }
        return acc;
    }
    // ... to the right-hand side of level LV - 1
    template <int LV> __device__ void restrict_to(const T (&v)[8])
    {
        const T acc = weighted<LV>(v);
        if constexpr (LV == 2) {
            f1 = acc;                             // of the last block's thread
        } else {
            Own<T, LV> &o = own<LV>();
            mem[at_f<LV - 1>() + o.ar] = acc;
            sync<LV>();
            if (mine<LV - 1>()) {
                constexpr int N = Lv<LV>::NQ;     // nodes 0 .. N - 1 of level LV - 1 in a row
                Own<T, LV - 1> &p = own<LV - 1>();
                p.fresh();
                const T *F = mem + at_f<LV - 1>() + 2 * ((p.qz * N + p.qy) * N + p.qx);
#pragma unroll
                for (int e = 0; e < 8; ++e) p.f[e] = F[(e & 1) + N * (e >> 1 & 1) + N * N * (e >> 2)];
            }
        }
    }
    template <int LV> __device__ void zero_below(int threads)   // u of level LV - 1
    {
        if constexpr (LV == 2) {
            if (threadIdx.x < 27) mem[kAtU1 + threadIdx.x] = T(0);
        } else {
            for (int p = threadIdx.x; p < 8 * Lv<LV - 1>::S; p += threads) mem[at_u<LV - 1>() + p] = T(0);
            Own<T, LV - 1> &p = own<LV - 1>();
#pragma unroll
            for (int e = 0; e < 8; ++e) p.u[e] = T(0);
        }
    }
    __device__ void exact()   // the 3^3 level's one interior node, by the last 5^3 block's thread
    {
#pragma clang fp contract(off)
        if (threadIdx.x == 7) {
            const T *v = mem + kAtU1;
            const double h = L / 2.0;
            const double s = double(v[12]) + double(v[14]) + double(v[10]) + double(v[16]) + double(v[4]) + double(v[22]);
            mem[kAtU1 + 13] = T((s - h * h * double(f1)) / 6.0);
        }
    }
    template <int LV> static __device__ int place(int i, int j, int k)   // of a node in LDS
    {
        if constexpr (LV == 1) return kAtU1 + i + 3 * (j + 3 * k);
        constexpr int NQ = Lv<LV>::NQ, Q = Lv<LV>::Q;
        const int q = i >> 1, row = (k >> 1) * Q + (j >> 1);
        return at_u<LV>() + ((i & 1) + 2 * (j & 1) + 4 * (k & 1)) * Lv<LV>::S + (q < NQ ? row * NQ + q : NQ * Q * Q + row);
    }
    // level LC -> LC + 1: the trilinear expression of the prolongation kernel, in
    // its order, without the terms of weight zero
    template <int LC> __device__ void prolong(bool add)
    {
#pragma clang fp contract(off)
        constexpr int LV = LC + 1;
        Own<T, LV> &o = own<LV>();
        o.fresh();
        T x[2][2][2];                             // [plane][row][column parity]: along x
#pragma unroll
        for (int z = 0; z < 2; ++z)
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                const T a = mem[place<LC>(o.qx, o.qy + y, o.qz + z)], b = mem[place<LC>(o.qx + 1, o.qy + y, o.qz + z)];
                x[z][y][0] = a;
                x[z][y][1] = T(0.5) * a + T(0.5) * b;
            }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int ex = e & 1;
            const T a = e & 2 ? T(0.5) * x[0][0][ex] + T(0.5) * x[0][1][ex] : x[0][0][ex];
            const T b = e & 2 ? T(0.5) * x[1][0][ex] + T(0.5) * x[1][1][ex] : x[1][0][ex];
            const T v = e & 4 ? T(0.5) * a + T(0.5) * b : a;
            o.u[e] = o.interior(e) ? (add ? o.u[e] + v : v) : o.u[e];
        }
        put_u<LV, 2>(o);
        sync<LV>();
    }
    template <int LV> __device__ void vcycle()
    {
        if constexpr (LV == 1) {
            exact();
            sync<1>();
        } else {
#pragma clang fp contract(off)
            sweeps<LV>(npre);
            Own<T, LV> &o = own<LV>();
            const T ih = ih2 * (T(1) / T(1 << 2 * (TOP - LV)));
            T r[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) r[e] = o.f[e] - (neighbours<LV>(o, e) - T(6) * o.u[e]) * ih;
            zero_below<LV>(LV >= 4 ? Lv<4>::OWN : 64);
            restrict_to<LV>(r);
            if (mine<LV - 1>()) vcycle<LV - 1>();
            if constexpr (LV >= 4) __syncthreads();
            prolong<LV - 1>(true);
            sweeps<LV>(npost);
        }
    }
    template <int LV> __device__ void restrict_all()   // f of the levels below LV
    {
        if constexpr (LV >= 2) {
            restrict_to<LV>(own<LV>().f);
            if (mine<LV - 1>()) restrict_all<LV - 1>();
        }
    }
    template <int LV> __device__ void inject()   // boundary of level LV from the top level, interior 0
    {
        constexpr int n = (1 << LV) + 1, st = 1 << (TOP - LV);
        for (int p = threadIdx.x; p < n * n * n; p += Lv<TOP>::OWN >= 64 ? Lv<TOP>::OWN : 64) {
            const int i = p % n, j = p / n % n, k = p / (n * n);
            const bool bnd = i == 0 || j == 0 || k == 0 || i == n - 1 || j == n - 1 || k == n - 1;
            mem[place<LV>(i, j, k)] = bnd ? mem[place<TOP>(i * st, j * st, k * st)] : T(0);
        }
        if constexpr (LV + 1 < TOP) inject<LV + 1>();
    }
    template <int LV> __device__ void load_below()   // the owners' u of the levels below LV from LDS
    {
        if constexpr (LV > 2) {
            Own<T, LV - 1> &o = own<LV - 1>();
#pragma unroll
            for (int e = 0; e < 8; ++e) o.u[e] = mem[at_u<LV - 1>() + o.at + e * Lv<LV - 1>::S];
            load_below<LV - 1>();
        }
    }
    template <int LV> __device__ void fmg_up(int ncycle)
    {
        if constexpr (LV <= TOP) {
            if (mine<LV>()) {
                prolong<LV - 1>(false);
                for (int c = 0; c < ncycle; ++c) vcycle<LV>();
            }
            if constexpr (LV == 3) __syncthreads();
            fmg_up<LV + 1>(ncycle);
        }
    }

    // mode 0: nrep V-cycles of the top level; 1: FMG; 2: one V-cycle from u = 0, not read
    __device__ void run(const T *fg, T *ug, int ncycle, int mode, int nrep)
    {
        typedef T pair_t __attribute__((ext_vector_type(2), aligned(sizeof(T))));
        constexpr int n = Lv<TOP>::n, NT = Lv<TOP>::OWN >= 64 ? Lv<TOP>::OWN : 64, NF = 3 * n * n;
        Own<T, TOP> &o = own<TOP>();
        const int g = 2 * (o.qx + n * (o.qy + n * o.qz));
        // node p of the three far faces
        auto far = [](int p, int &i, int &j, int &k) {
            const int d = p / (n * n), a = p % n, b = p / n % n;
            i = d == 0 ? n - 1 : a;
            j = d == 0 ? a : d == 1 ? n - 1 : b;
            k = d == 2 ? n - 1 : b;
        };
        pair_t fv[4], uv[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int p = g + n * ((r & 1) + n * (r >> 1));
            fv[r] = *reinterpret_cast<const pair_t *>(fg + p);
            uv[r] = mode == 2 ? pair_t{T(0), T(0)} : *reinterpret_cast<const pair_t *>(ug + p);
        }
        for (int p = threadIdx.x; p < NF; p += NT) {
            int i, j, k;
            far(p, i, j, k);
            mem[place<TOP>(i, j, k)] = mode == 2 ? T(0) : ug[i + n * (j + n * k)];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            o.f[2 * r] = fv[r].x;
            o.f[2 * r + 1] = fv[r].y;
            o.u[2 * r] = uv[r].x;
            o.u[2 * r + 1] = uv[r].y;
        }
        put_u<TOP, 2>(o);
        __syncthreads();
        if (mode == 1) {
            restrict_all<TOP>();
            inject<1>();
            __syncthreads();
            load_below<TOP>();
            exact();
            __syncthreads();
            fmg_up<2>(ncycle);
        } else {
            for (int c = 0; c < nrep; ++c) vcycle<TOP>();
        }
        if (o.act) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                *reinterpret_cast<pair_t *>(ug + g + n * ((r & 1) + n * (r >> 1))) = pair_t{o.u[2 * r], o.u[2 * r + 1]};
        }
        if (mode == 2)
            for (int p = threadIdx.x; p < NF; p += NT) {
                int i, j, k;
                far(p, i, j, k);
                ug[i + n * (j + n * k)] = T(0);
            }
    }
};

template <typename T, int TOP>
__global__ void __launch_bounds__(Lv<TOP>::OWN >= 64 ? Lv<TOP>::OWN : 64)
coarse_tail_k(double L, T h2, T ih2, const T *__restrict__ fg, T *__restrict__ ug, int npre, int npost, int ncycle,
              int mode, int nrep)
{
    __shared__ T mem[kTailLds];
    Tail<T, TOP> t{mem, L, h2, ih2, npre, npost, {}, {}, {}, T(0)};
    t.o4.init();
    t.o3.init();
    t.o2.init();
    constexpr int n = Lv<TOP>::n;
    t.run(fg + (size_t)blockIdx.x * n * n * n, ug + (size_t)blockIdx.x * n * n * n, ncycle, mode, nrep);
}

}  // namespace

template <typename T>
void launch_coarse_tail(int ltop, double L, const T *f, T *u, int npre, int npost, int ncycle, int mode, int nrep,
                        hipStream_t s, int nb)
{
    const T h = T(L) / T(1 << ltop), h2 = h * h, ih2 = T(1) / (h * h);
    const double Lt = double(T(L));
    auto go = [&](auto *kernel, int threads) {
        hipLaunchKernelGGL(kernel, dim3(nb), dim3(threads), 0, s, Lt, h2, ih2, f, u, npre, npost, ncycle, mode, nrep);
    };
    if (ltop >= kTailTop) go(coarse_tail_k<T, 4>, Lv<4>::OWN);
    else if (ltop == 3) go(coarse_tail_k<T, 3>, Lv<3>::OWN);
    else go(coarse_tail_k<T, 2>, 64);
}

template void launch_coarse_tail<double>(int, double, const double *, double *, int, int, int, int, int, hipStream_t, int);
template void launch_coarse_tail<float>(int, double, const float *, float *, int, int, int, int, int, hipStream_t, int);

}  // namespace qm
