// The coarse tail of the multigrid solves (Sec. 2 of Angus et al.): every level
// with at most 17 points per side inside one workgroup, so that a V-cycle or a
// whole FMG over these levels is one launch.  Level l has 2^l + 1 points; the
// 3^3 level is solved exactly, in FP64.
//
// A thread owns an x-pair of neighbouring nodes of a level (one red, one black:
// i + j + k even and odd; at 17^3 the pair on two neighbouring planes) and keeps
// its u and f in registers for the whole launch, on every level at once.  In
// LDS each level has an array per colour, [k][j][pair]: a colour pass reads only
// the other colour, at consecutive places, and only the neighbours the thread
// does not own (four of six at 17^3).  The residual is staged with even and odd
// columns apart, which is how the restriction reads it, and the prolongation
// takes the eight coarse values of a pair once for all its nodes.  17^3 has 960
// owners, 9^3 196; 5^3 and 3^3 fit one wavefront, which works through them on its
// own, in order and without barriers, while the others wait at one.
//
// Bound by the latency of its dependent phases (26 barriers per V-cycle from
// 17^3).  The form before this one held u, f and the residual in LDS in grid
// order and read seven values per node update at a stride of two, about twice
// the LDS cycles in conflicts; every phase had all 1024 threads meet at a
// barrier (34 per V-cycle).  Same operations in the same order.  A V-cycle from
// 17^3 14.4 -> 12.1 us (from 9^3 5.1 -> 5.0, from 5^3 2.0), a launch of one in a
// 65^3 step 26.8 -> 23.1 us on average.
#include "common.h"

namespace qm {

namespace {

constexpr int kTailTop = 4;
constexpr int kTailThreads = 1024;

template <int LV>
struct Lv {
    static constexpr int n = (1 << LV) + 1, m = n - 2;
    static constexpr int Q = (1 << (LV - 1)) + 1;        // pairs of a row, the far face's among them
    static constexpr int NQ = 1 << (LV - 1);             // ... that hold interior nodes: columns 2q, 2q + 1
    static constexpr int KB = LV == 4 ? 2 : 1;           // planes per owner
    static constexpr int G = (m + KB - 1) / KB, OWN = NQ * m * G;
    static constexpr int S = n * n * Q;                  // nodes of one colour, with the places no node has
    static_assert(OWN <= kTailThreads, "one owner per thread");
};

template <typename T>
struct TailShared {
    T u4[2][Lv<4>::S], u3[2][Lv<3>::S], u2[2][Lv<2>::S], u1[27];
    T r4[2 * Lv<4>::S], r3[2 * Lv<3>::S], r2[2 * Lv<2>::S];   // [k][j][parity of i][i / 2]
    T h2[kTailTop + 1], ih2[kTailTop + 1];
};

template <typename T, int LV>
struct Own {
    T u[2][Lv<LV>::KB], f[2][Lv<LV>::KB];    // by colour
    int q, j, k;                             // pair, row, first plane
    bool act;

    __device__ void init()
    {
        act = (int)threadIdx.x < Lv<LV>::OWN;
        const int t = act ? (int)threadIdx.x : 0;
        q = t % Lv<LV>::NQ;
        j = 1 + t / Lv<LV>::NQ % Lv<LV>::m;
        k = 1 + t / (Lv<LV>::NQ * Lv<LV>::m) * Lv<LV>::KB;
    }
    // The indices count as new from here: addresses of every phase kept across the cycles would spill.
    __device__ void fresh() { asm volatile("" : "+v"(q), "+v"(j), "+v"(k)); }
    __device__ int place(int kb) const { return ((k + kb) * Lv<LV>::n + j) * Lv<LV>::Q + q; }
    // which node of the pair has colour c on plane k + kb
    __device__ int node(int kb, int c) const { return ((j + k + kb) & 1) ^ c; }
    __device__ bool interior(int kb, int e) const { return act && (q > 0 || e) && k + kb <= Lv<LV>::m; }
};

template <typename T>
struct Tail {
    TailShared<T> &S;
    T L;
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
    template <int LV> __device__ T *u(int c)
    {
        if constexpr (LV == 4) return S.u4[c];
        else if constexpr (LV == 3) return S.u3[c];
        else return S.u2[c];
    }
    template <int LV> __device__ T *r()
    {
        if constexpr (LV == 4) return S.r4;
        else if constexpr (LV == 3) return S.r3;
        else return S.r2;
    }
    // Levels up to 5^3 belong to the first wavefront, whose LDS operations complete in order.
    template <int LV> __device__ void sync()
    {
        if constexpr (LV >= 3) {
            __syncthreads();
        } else {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    }
    template <int LV> __device__ static bool mine() { return LV >= 3 || threadIdx.x < 64; }

    // sum of the six neighbours of the node of colour c on plane k + kb, in grid order (the two of x commute)
    template <int LV> __device__ T neighbours(const Own<T, LV> &o, int kb, int c)
    {
#pragma clang fp contract(off)
        constexpr int Q = Lv<LV>::Q, P = Lv<LV>::n * Q, KB = Lv<LV>::KB;
        const T *O = u<LV>(c ^ 1) + o.place(kb);
        const T zm = kb == 0 ? O[-P] : o.u[c ^ 1][kb == 0 ? 0 : kb - 1];
        const T zp = kb == KB - 1 ? O[P] : o.u[c ^ 1][kb == KB - 1 ? kb : kb + 1];
        return o.u[c ^ 1][kb] + O[o.node(kb, c) ? 1 : -1] + O[-Q] + O[Q] + zm + zp;
    }
    template <int LV> __device__ void pass(int c)
    {
#pragma clang fp contract(off)
        Own<T, LV> &o = own<LV>();
        const T hh = S.h2[LV], sixth = T(1) / T(6);
        o.fresh();
        if (o.act) {
            T v[Lv<LV>::KB];
#pragma unroll
            for (int kb = 0; kb < Lv<LV>::KB; ++kb) v[kb] = (neighbours<LV>(o, kb, c) - hh * o.f[c][kb]) * sixth;
#pragma unroll
            for (int kb = 0; kb < Lv<LV>::KB; ++kb)
                if (o.interior(kb, o.node(kb, c))) {
                    o.u[c][kb] = v[kb];
                    u<LV>(c)[o.place(kb)] = v[kb];
                }
        }
        sync<LV>();
    }
    template <int LV> __device__ void sweeps(int ns)
    {
        for (int s = 0; s < ns; ++s) {
            pass<LV>(0);
            pass<LV>(1);
        }
    }
    // values of the owner's interior nodes into the staging array of level LV
    template <int LV, typename V> __device__ void stage(V value)
    {
        Own<T, LV> &o = own<LV>();
        o.fresh();
#pragma unroll
        for (int kb = 0; kb < Lv<LV>::KB; ++kb)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int e = o.node(kb, c);
                if (o.interior(kb, e))
                    r<LV>()[(((o.k + kb) * Lv<LV>::n + o.j) * 2 + e) * Lv<LV>::Q + o.q] = value(o, kb, c);
            }
    }
    template <int LV> __device__ void residual()   // staged; and the next level's u becomes zero
    {
        const T ih = S.ih2[LV];
        stage<LV>([&](const Own<T, LV> &o, int kb, int c) {
#pragma clang fp contract(off)
            return o.f[c][kb] - (neighbours<LV>(o, kb, c) - T(6) * o.u[c][kb]) * ih;
        });
        constexpr int NT = LV >= 3 ? kTailThreads : 64;
        if constexpr (LV == 2) {
            if (threadIdx.x < 27) S.u1[threadIdx.x] = T(0);
        } else {
            T *z = u<LV - 1>(0);
            for (int p = threadIdx.x; p < 2 * Lv<LV - 1>::S; p += NT) z[p] = T(0);
        }
        sync<LV>();
    }
    // full weighting of the staged values of level LV at its coarse node (I, J, K)
    template <int LV> __device__ T weighted(int I, int J, int K)
    {
#pragma clang fp contract(off)
        constexpr int n = Lv<LV>::n, Q = Lv<LV>::Q;
        const T w[3] = {T(0.25), T(0.5), T(0.25)};
        T acc = T(0);
#pragma unroll
        for (int c = -1; c <= 1; ++c) {
            T v[9];
#pragma unroll
            for (int b = -1; b <= 1; ++b)
#pragma unroll
                for (int a = -1; a <= 1; ++a)
                    v[(a + 1) + 3 * (b + 1)] = r<LV>()[(((2 * K + c) * n + 2 * J + b) * 2 + (a & 1)) * Q + (a < 0 ? I - 1 : I)];
#pragma unroll
            for (int b = -1; b <= 1; ++b)
#pragma unroll
                for (int a = -1; a <= 1; ++a) acc += (w[a + 1] * w[b + 1] * w[c + 1]) * v[(a + 1) + 3 * (b + 1)];
        }
        return acc;
    }
    template <int LV> __device__ void restrict_to()   // f of level LV - 1, its owners' u zero
    {
        if constexpr (LV == 2) {
            if (threadIdx.x == 0) f1 = weighted<2>(1, 1, 1);
        } else {
            Own<T, LV - 1> &o = own<LV - 1>();
            o.fresh();
#pragma unroll
            for (int kb = 0; kb < Lv<LV - 1>::KB; ++kb)
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const int e = o.node(kb, c);
                    o.u[c][kb] = T(0);
                    o.f[c][kb] = o.interior(kb, e) ? weighted<LV>(2 * o.q + e, o.j, o.k + kb) : T(0);
                }
        }
    }
    __device__ void exact()   // the 3^3 level's one interior node, by the first thread
    {
#pragma clang fp contract(off)
        if (threadIdx.x == 0) {
            const T *v = S.u1;
            const double h = double(L) / 2.0;
            const double s = double(v[12]) + double(v[14]) + double(v[10]) + double(v[16]) + double(v[4]) + double(v[22]);
            S.u1[13] = T((s - h * h * double(f1)) / 6.0);
        }
    }
    template <int LC> __device__ T coarse(int I, int J, int K)
    {
        if constexpr (LC == 1) return S.u1[I + 3 * (J + 3 * K)];
        else return u<LC>((I + J + K) & 1)[(K * Lv<LC>::n + J) * Lv<LC>::Q + (I >> 1)];
    }
    // level LC -> LC + 1: the trilinear expression of the prolongation kernel, in its order
    template <int LC> __device__ void prolong(bool add)
    {
#pragma clang fp contract(off)
        constexpr int LV = LC + 1, KB = Lv<LV>::KB;
        Own<T, LV> &o = own<LV>();
        o.fresh();
        if (o.act) {
            const int ja = o.j >> 1, jb = (o.j + 1) >> 1, dj = o.j & 1;
            const T wja = dj ? T(0.5) : T(1), wjb = dj ? T(0.5) : T(0);
            T row[2][2][2];              // [coarse plane k / 2, (k + 1) / 2 of the first plane][row a, b][column q, q + 1]
            const int pl[2] = {o.k >> 1, (o.k + 1) >> 1};
#pragma unroll
            for (int z = 0; z < 2; ++z)
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    row[z][0][x] = coarse<LC>(o.q + x, ja, pl[z]);
                    row[z][1][x] = coarse<LC>(o.q + x, jb, pl[z]);
                }
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                // with two planes the first is odd and the second, even, lies on the upper coarse plane
                const bool ko = KB == 2 ? kb == 0 : (o.k & 1);
                const T wka = ko ? T(0.5) : T(1), wkb = ko ? T(0.5) : T(0);
                const int za = KB == 2 && kb == 1 ? 1 : 0;
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const int e = o.node(kb, c);
                    auto along_x = [&](const T *p) {
                        return (e ? T(0.5) : T(1)) * p[0] + (e ? T(0.5) : T(0)) * (e ? p[1] : p[0]);
                    };
                    const T xa = along_x(row[za][0]), xb = along_x(row[za][1]), xc = along_x(row[1][0]),
                            xd = along_x(row[1][1]);
                    const T v = wka * (wja * xa + wjb * xb) + wkb * (wja * xc + wjb * xd);
                    if (o.interior(kb, e)) {
                        o.u[c][kb] = add ? o.u[c][kb] + v : v;
                        u<LV>(c)[o.place(kb)] = o.u[c][kb];
                    }
                }
            }
        }
        sync<LV>();
    }
    template <int LV> __device__ void vcycle()
    {
        if constexpr (LV == 1) {
            exact();
            sync<1>();
        } else {
            sweeps<LV>(npre);
            residual<LV>();
            if constexpr (LV == 3) {     // the first wavefront alone below 9^3
                if (mine<2>()) {
                    restrict_to<3>();
                    vcycle<2>();
                }
                __syncthreads();
            } else {
                restrict_to<LV>();
                vcycle<LV - 1>();
            }
            prolong<LV - 1>(true);
            sweeps<LV>(npost);
        }
    }
    template <int LV> __device__ void restrict_all()   // f of the levels below LV, by all threads
    {
        if constexpr (LV >= 2) {
            stage<LV>([](const Own<T, LV> &o, int kb, int c) { return o.f[c][kb]; });
            __syncthreads();
            restrict_to<LV>();
            restrict_all<LV - 1>();
        }
    }
    template <int LV> __device__ void load_own()   // the owners' u from LDS
    {
        Own<T, LV> &o = own<LV>();
#pragma unroll
        for (int kb = 0; kb < Lv<LV>::KB; ++kb)
#pragma unroll
            for (int c = 0; c < 2; ++c) o.u[c][kb] = u<LV>(c)[o.place(kb)];
    }
    template <int LV, int TOP> __device__ void inject()   // boundary of level LV from level TOP, interior 0
    {
        constexpr int n = (1 << LV) + 1, st = 1 << (TOP - LV);
        for (int p = threadIdx.x; p < n * n * n; p += kTailThreads) {
            const int i = p % n, j = p / n % n, k = p / (n * n);
            const bool bnd = i == 0 || j == 0 || k == 0 || i == n - 1 || j == n - 1 || k == n - 1;
            const T v = bnd ? coarse<TOP>(i * st, j * st, k * st) : T(0);
            if constexpr (LV == 1) S.u1[p] = v;
            else u<LV>((i + j + k) & 1)[(k * n + j) * Lv<LV>::Q + (i >> 1)] = v;
        }
    }
    template <int LV, int TOP> __device__ void inject_all()
    {
        if constexpr (LV < TOP) {
            inject<LV, TOP>();
            inject_all<LV + 1, TOP>();
        }
    }
    template <int LV, int TOP> __device__ void load_all()
    {
        if constexpr (LV < TOP) {
            load_own<LV>();
            load_all<LV + 1, TOP>();
        }
    }
    template <int LV, int TOP> __device__ void fmg_up(int ncycle)
    {
        if constexpr (LV <= TOP) {
            if (mine<LV>()) {
                prolong<LV - 1>(false);
                for (int c = 0; c < ncycle; ++c) vcycle<LV>();
            }
            if constexpr (LV == 2) __syncthreads();
            fmg_up<LV + 1, TOP>(ncycle);
        }
    }

    // mode 0: nrep V-cycles of the top level; 1: FMG; 2: one V-cycle from u = 0, not read
    template <int TOP> __device__ void run(const T *fg, T *ug, int ncycle, int mode, int nrep)
    {
        constexpr int n = Lv<TOP>::n, cnt = n * n * n, NL = (cnt + kTailThreads - 1) / kTailThreads;
        Own<T, TOP> &o = own<TOP>();
        // all global loads of a thread first
        T x[NL];
#pragma unroll
        for (int t = 0; t < NL; ++t) x[t] = mode == 2 ? T(0) : ug[min((int)threadIdx.x + t * kTailThreads, cnt - 1)];
#pragma unroll
        for (int kb = 0; kb < Lv<TOP>::KB; ++kb)
#pragma unroll
            for (int c = 0; c < 2; ++c)
                o.f[c][kb] = fg[2 * o.q + o.node(kb, c) + n * (o.j + n * (o.k + kb))];
#pragma unroll
        for (int t = 0; t < NL; ++t) {
            const int p = threadIdx.x + t * kTailThreads;
            const int i = p % n, j = p / n % n, k = p / (n * n);
            if (p < cnt) u<TOP>((i + j + k) & 1)[(k * n + j) * Lv<TOP>::Q + (i >> 1)] = x[t];
        }
        __syncthreads();
        load_own<TOP>();
        if (mode == 1) {
            restrict_all<TOP>();
            inject_all<1, TOP>();
            __syncthreads();
            load_all<2, TOP>();
            exact();
            __syncthreads();
            fmg_up<2, TOP>(ncycle);
        } else if (mine<TOP>()) {
            for (int c = 0; c < nrep; ++c) vcycle<TOP>();
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < NL; ++t) {
            const int p = threadIdx.x + t * kTailThreads;
            if (p < cnt) ug[p] = coarse<TOP>(p % n, p / n % n, p / (n * n));
        }
    }
};

template <typename T>
__global__ void __launch_bounds__(kTailThreads)
coarse_tail_k(int top, T L, const T *__restrict__ fg, T *__restrict__ ug, int npre, int npost, int ncycle, int mode,
              int nrep)
{
    __shared__ TailShared<T> S;
    Tail<T> t{S, L, npre, npost, {}, {}, {}, T(0)};
    t.o4.init();
    t.o3.init();
    t.o2.init();
    if (threadIdx.x == 0) {
        for (int l = 1; l <= kTailTop; ++l) {
            const T h = L / T((1 << l));
            S.h2[l] = h * h;
            S.ih2[l] = T(1) / (h * h);
        }
    }
    const int n = (1 << top) + 1;
    fg += (size_t)blockIdx.x * n * n * n;
    ug += (size_t)blockIdx.x * n * n * n;
    switch (top) {
    case 2: t.template run<2>(fg, ug, ncycle, mode, nrep); break;
    case 3: t.template run<3>(fg, ug, ncycle, mode, nrep); break;
    default: t.template run<4>(fg, ug, ncycle, mode, nrep); break;
    }
}

}  // namespace

template <typename T>
void launch_coarse_tail(int ltop, double L, const T *f, T *u, int npre, int npost, int ncycle, int mode, int nrep,
                        hipStream_t s, int nb)
{
    hipLaunchKernelGGL(coarse_tail_k<T>, dim3(nb), dim3(kTailThreads), 0, s, ltop, T(L), f, u, npre, npost, ncycle,
                       mode, nrep);
}

template void launch_coarse_tail<double>(int, double, const double *, double *, int, int, int, int, int, hipStream_t, int);
template void launch_coarse_tail<float>(int, double, const float *, float *, int, int, int, int, int, hipStream_t, int);

}  // namespace qm
