// Kernels of the 3D U-Net that predicts the QUMOND potential from (Phi_N,
// source) as an initial guess for the second multigrid solve.
//
// Tensors are channel-last BF16 on vertex-centred n^3 grids: element (v, c)
// of a tensor with slot width `cs` sits at v * cs + c (v = i + n (j + n k)), so
// a tensor can be a channel slice of a wider one (skip connections are
// written straight into the concatenated input of the decoder convolution).
// Slot widths and channel offsets are multiples of 8 (16-byte fragments).
//
// Convolutions are implicit GEMMs on v_mfma_f32_16x16x32_bf16 with FP32
// accumulation: rows = 16 output voxels, columns = 16 output channels,
// K = 27 taps x input channels (padded to a multiple of 32).  With the lane
// layout of that instruction, lane l supplies row/column l % 16 and the
// eight consecutive K indices 8 (l / 16) .. 8 (l / 16) + 7, which are eight
// consecutive channels of one tap: one 16-byte load.  The 4 accumulators of
// lane l are column l % 16, rows 4 (l / 16) + r.
#include <type_traits>

#include "common.h"
#include "unet.h"

namespace qm {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

__device__ __forceinline__ void decode3(int v, int n, int &i, int &j, int &k)
{
    i = v % n;
    const int t = v / n;
    j = t % n;
    k = t / n;
}

// ------------------------------------------------------------ convolution

// y[v, co] = act(bias[co] + sum_{tap, ci} x[s v + d(tap), ci] W[co, tap cin + ci])
//
// Each wave computes RB blocks of 16 consecutive output voxels for all cout
// = 16 NB channels: per K-chunk it loads RB activation fragments and NB weight
// fragments and issues RB x NB MFMAs, and it loads the next chunk's fragments
// before the current chunk's MFMAs.  Every output is accumulated over the
// K-chunks in the same order whatever RB is.
template <int NB, int RB>
__global__ void __launch_bounds__(256)
conv3d_fwd_k(Tensor x, int cin, const __bf16 *__restrict__ wt, int kpad, const float *__restrict__ bias, Tensor y,
             int stride, int relu)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nout = y.n, nin = x.n;
    const int Nout = nout * nout * nout;
    const int v0 = (blockIdx.x * 4 + wave) * 16 * RB;
    if (v0 >= Nout) return;
    const int g = lane >> 4, r16 = lane & 15;
    int bi[RB], bj[RB], bk[RB];
    bool ok[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int va = v0 + 16 * rb + r16;
        int io = 0, jo = 0, ko = 0;
        ok[rb] = va < Nout;
        if (ok[rb]) decode3(va, nout, io, jo, ko);
        bi[rb] = stride * io;
        bj[rb] = stride * jo;
        bk[rb] = stride * ko;
    }
    const int kreal = 27 * cin;
    const size_t xcs = (size_t)x.cs;
    // K index of this lane's fragment in the current chunk, as (tap, channel)
    int kk0 = 8 * g, tap = kk0 / cin, c0 = kk0 - tap * cin;
    auto load = [&](bf16x8 *a, bf16x8 *w) {
        const bool live = kk0 < kreal;
        const int di = tap % 3 - 1, dj = (tap / 3) % 3 - 1, dk = tap / 9 - 1;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            bf16x8 t = {};
            const int i = bi[rb] + di, j = bj[rb] + dj, k = bk[rb] + dk;
            if (live && ok[rb] && i >= 0 && i < nin && j >= 0 && j < nin && k >= 0 && k < nin)
                t = *reinterpret_cast<const bf16x8 *>(x.p + (size_t)(i + nin * (j + nin * k)) * xcs + c0);
            a[rb] = t;
        }
#pragma unroll
        for (int b = 0; b < NB; ++b)
            w[b] = *reinterpret_cast<const bf16x8 *>(wt + (size_t)(b * 16 + r16) * kpad + kk0);
        kk0 += 32;
        c0 += 32;
        while (c0 >= cin) {
            c0 -= cin;
            ++tap;
        }
    };
    f32x4 acc[RB][NB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[rb][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 a[RB], w[NB];
    load(a, w);
    for (int kc = 0; kc < kpad; kc += 32) {
        bf16x8 an[RB], wn[NB];
        if (kc + 32 < kpad) load(an, wn);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[rb][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[rb], w[b], acc[rb][b], 0, 0, 0);
        if (kc + 32 < kpad) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) a[rb] = an[rb];
#pragma unroll
            for (int b = 0; b < NB; ++b) w[b] = wn[b];
        }
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int co = b * 16 + r16;
        const float bb = bias ? bias[co] : 0.f;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int v = v0 + 16 * rb + 4 * g + r;
                if (v >= Nout) continue;
                float val = acc[rb][b][r] + bb;
                if (relu) val = val > 0.f ? val : 0.f;
                y.p[(size_t)v * y.cs + co] = (__bf16)val;
            }
    }
}

// Stride-1 convolution with the input tile in LDS: a workgroup computes a
// 16 x 4 x 4 block of output voxels (each wave 4 x-rows of 16 voxels, one
// MFMA column block each) for 16 NB output channels (blockIdx.y picks them).  The
// input channels are taken in chunks of 32 and a rest of 16 or 8; for each chunk
// the 18 x 6 x 6 input voxels (block plus a one-voxel ring) are staged in LDS
// once and every one of the 27 taps reads its activation fragments from there.
// Within a chunk of cc channels the K-steps of 32 cover 32 / cc taps at a time,
// in the same (tap, channel) order as conv3d_fwd_k.
//
// What bounds it is latency, then the LDS reads (one per MFMA at 16 output channels):
// all loads of a chunk are in flight at once (a loop of load and store had waited
// for each of its ten loads in turn); weights come a tap or a group of taps ahead,
// or stay in registers (16 and 8 input channels); and output channels are the rows
// of the product, so a lane stores four of them at once.  NB blocks of 16 output
// channels share a staged tile.
//
// AHEAD: a workgroup takes a run of tiles and loads the next chunk or tile during
// the MFMAs of this one.  That pays with 8, 16 and 48 input channels.  In whole
// chunks of 32 the registers of those loads cost a wavefront per SIMD, which is
// worth more: a tile per workgroup, NB up to 4 (32 -> 32 channels at 97^3 with runs
// 105 us at best, without 93; 64 -> 64 531 and 492; 96 -> 32 358 and 277).
//
// The first form, one tile per workgroup for all channels with every load waited for
// -> now, same bits: 48 -> 16 channels at 129^3 417 -> 210 us, 16 -> 16 180 -> 87, 8 -> 16
// 104 -> 49, 96 -> 32 at 65^3 151 -> 99, 32 -> 64 at 97^3 217 -> 166, 64 -> 64 512 -> 492.
constexpr int kTileX = 16, kTileY = 4, kTileZ = 4;
constexpr int kInX = kTileX + 2, kInY = kTileY + 2, kInZ = kTileZ + 2, kInV = kInX * kInY * kInZ;

template <int NB, int C0, bool AHEAD>
__global__ void __launch_bounds__(256, AHEAD && C0 == 32 && NB > 1 ? 2 : 3)
conv3d_fwd_lds_k(Tensor x, int cin, const __bf16 *__restrict__ wt, int kpad, const float *__restrict__ bias, Tensor y,
                 int relu, int tx, int ty, int tiles, int per)
{
    constexpr int RB = 4;
    constexpr int Q = C0 / 8, VS = 256 / Q, NL = (kInV + VS - 1) / VS;   // NL 16-byte loads per thread and chunk
    constexpr int kPitch = C0 == 8 ? 8 : C0 + 8;   // bf16 per staged voxel (padded against bank conflicts)
    __shared__ __attribute__((aligned(16))) __bf16 tile[kInV * kPitch];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int g = lane >> 4, r16 = lane & 15;
    const int n = y.n;   // = x.n (stride 1)
    const int co0 = blockIdx.y * 16 * NB;
    wt += (size_t)co0 * kpad;
    int t = (int)xcd_tile(blockIdx.x, gridDim.x) * per;      // this workgroup's run of tiles
    const int tend = min(tiles, t + per);
    if (t >= tend) return;

    // Staging: in round r this thread takes 8 channels (q) of voxel v0 + VS r;
    // from clamped addresses, zeroed where it is stored outside the grid.
    const int q = threadIdx.x % Q, v0 = threadIdx.x / Q;
    unsigned okp = 0;
    auto origin = [&](int tt, int &X0, int &Y0, int &Z0) {
        X0 = tt % tx * kTileX;
        Y0 = tt / tx % ty * kTileY;
        Z0 = tt / tx / ty * kTileZ;
    };
    bf16x8 pre[NL];
    auto fetch = [&](int tt, int cb) {
        int X0, Y0, Z0;
        origin(tt, X0, Y0, Z0);
        // a rest of 16 or 8 channels: the other q load it again, unused
        const __bf16 *src = x.p + min(cb + 8 * q, cin - 8);
        okp = 0;
        int vb = v0;
        asm volatile("" : "+v"(vb));     // decoded anew for every tile: kept across them the decodings would spill
#pragma unroll
        for (int r = 0; r < NL; ++r) {
            const int v = vb + VS * r;
            const int i = X0 - 1 + v % kInX, j = Y0 - 1 + v / kInX % kInY, k = Z0 - 1 + v / (kInX * kInY);
            const bool in = v < kInV && i >= 0 && i < n && j >= 0 && j < n && k >= 0 && k < n;
            pre[r] = *reinterpret_cast<const bf16x8 *>(src + (size_t)(in ? i + n * (j + n * k) : 0) * x.cs);
            okp |= (unsigned)in << r;
        }
    };
    auto commit = [&]() {
#pragma unroll
        for (int r = 0; r < NL; ++r)
            if (v0 + VS * r < kInV)
                *reinterpret_cast<bf16x8 *>(tile + (v0 + VS * r) * kPitch + 8 * q) = (okp >> r) & 1 ? pre[r] : bf16x8{};
    };
    f32x4 acc[RB][NB];
    // this lane's rows: wave w, row block rb -> output row (y, z) = (rb, w) of the block, x = r16
    const __bf16 *mine = tile + (r16 + kInX * kInY * wave) * kPitch;
    const __bf16 *wrow = wt + (size_t)r16 * kpad;
    auto frag = [&](const __bf16 *p) { return *reinterpret_cast<const bf16x8 *>(p); };
    auto mac = [&](int rb, const bf16x8 &a, const bf16x8 *w) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
            acc[rb][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[b], a, acc[rb][b], 0, 0, 0);
    };
    // 32 channels, one tap per K-step: the three dx of an input row are read once
    // per dz and serve the (up to three) dy that meet it
    auto chunk32 = [&](int cb) {
        const __bf16 *wp = wrow + cb + 8 * g;
        auto weights = [&](int row, bf16x8 (*w)[NB]) {   // the three taps of row = dy + 3 dz
#pragma unroll
            for (int e = 0; e < 3; ++e)
#pragma unroll
                for (int b = 0; b < NB; ++b) w[e][b] = frag(wp + (size_t)(b * 16) * kpad + (3 * row + e) * cin);
        };
        bf16x8 w[2][3][NB];
        weights(0, w[0]);
#pragma unroll 1
        for (int dz = 0; dz < 3; ++dz) {
            const __bf16 *p = mine + kInX * kInY * dz * kPitch + 8 * g;
            bf16x8 a[RB + 2][3];
#pragma unroll
            for (int y = 0; y < RB; ++y)
#pragma unroll
                for (int e = 0; e < 3; ++e) a[y][e] = frag(p + (e + kInX * y) * kPitch);
#pragma unroll
            for (int dy = 0; dy < 3; ++dy) {
                weights(min(3 * dz + dy + 1, 8), w[(dy + 1) & 1]);
                if (dy < 2)
#pragma unroll
                    for (int e = 0; e < 3; ++e) a[RB + dy][e] = frag(p + (e + kInX * (RB + dy)) * kPitch);
#pragma unroll
                for (int e = 0; e < 3; ++e)
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) mac(rb, a[rb + dy][e], w[dy & 1][e]);
            }
#pragma unroll
            for (int e = 0; e < 3; ++e)
#pragma unroll
                for (int b = 0; b < NB; ++b) w[0][e][b] = w[1][e][b];
        }
    };
    // ... a tap at a time, its rows and weights one tap ahead, in a third of the registers
    auto chunk32_taps = [&](int cb) {
        const __bf16 *wp = wrow + cb + 8 * g;
        auto weights = [&](int tap, bf16x8 *w) {
#pragma unroll
            for (int b = 0; b < NB; ++b) w[b] = frag(wp + (size_t)(b * 16) * kpad + tap * cin);
        };
        auto rows = [&](const __bf16 *p, int t, bf16x8 *a) {   // of tap t = dx + 3 dy
#pragma unroll
            for (int y = 0; y < RB; ++y) a[y] = frag(p + (t % 3 + kInX * (t / 3 + y)) * kPitch);
        };
        bf16x8 w[2][NB], a[2][RB];
        weights(0, w[0]);
#pragma unroll 1
        for (int dz = 0; dz < 3; ++dz) {
            const __bf16 *p = mine + kInX * kInY * dz * kPitch + 8 * g;
            rows(p, 0, a[0]);
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                if (t < 8) rows(p, t + 1, a[(t + 1) & 1]);
                weights(min(9 * dz + t + 1, 26), w[(t + 1) & 1]);
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) mac(rb, a[t & 1][rb], w[t & 1]);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int b = 0; b < NB; ++b) w[0][b] = w[1][b];     // nine taps, two sets
        }
    };
    // 16 or 8 channels: 2 or 4 taps per K-step, by the lane's quarter; the last
    // step's taps beyond 26 count as zeros
    auto chunk_small = [&](auto CC, int cb, auto &&weight) {
        constexpr int cc = CC.value, TAPS = 32 / cc, STEPS = (27 * cc + 31) / 32;
        const int sub = (8 * g) / cc, cl = (8 * g) % cc;        // this lane's tap of a step and its channels
        bf16x8 w[3][NB];                                        // of this step and the next two
        weight(0, w[0]);
        weight(1, w[1]);
#pragma unroll
        for (int st = 0; st < STEPS; ++st) {
            const bool last = TAPS * (st + 1) > 27;
            const bool live = !last || TAPS * st + sub < 27;
            int to = 0;
#pragma unroll
            for (int u = 0; u < TAPS; ++u) {
                const int tap = min(TAPS * st + u, 26);
                const int o = (tap % 3 + kInX * (tap / 3 % 3 + kInY * (tap / 9))) * kPitch;
                to = sub == u ? o : to;
            }
            if (st + 2 < STEPS) weight(st + 2, w[(st + 2) % 3]);
            if (last && !live) {
#pragma unroll
                for (int b = 0; b < NB; ++b) w[st % 3][b] = bf16x8{};
            }
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                bf16x8 a = frag(mine + to + cl + kInX * rb * kPitch);
                if (last && !live) a = bf16x8{};
                mac(rb, a, w[st % 3]);
            }
            __builtin_amdgcn_sched_barrier(0);   // keep the reads of later steps from piling up in registers
        }
    };
    // weights of a small chunk from memory, each step's before its reads
    auto from_memory = [&](auto CC, int cb) {
        constexpr int cc = CC.value, TAPS = 32 / cc;
        int first = (8 * g) / cc * cin + cb + (8 * g) % cc;
        asm volatile("" : "+v"(first));      // addresses from here: kept across tiles they would spill
        return [=](int st, bf16x8 *w) {
            const int at = min(first + st * TAPS * cin, kpad - 8);   // the last step's dead taps stay in the row
#pragma unroll
            for (int b = 0; b < NB; ++b) w[b] = *reinterpret_cast<const bf16x8 *>(wrow + b * 16 * kpad + at);
        };
    };
    // ... of a layer of 16 or 8 input channels in registers, for the whole run of tiles
    constexpr int KS = C0 == 32 ? 1 : (27 * C0 + 31) / 32;
    constexpr bool KEEP = C0 < 32 && KS * NB <= 14;
    bf16x8 kept[KEEP ? KS : 1][NB];
    if constexpr (KEEP) {
        auto get = from_memory(std::integral_constant<int, C0>{}, 0);
#pragma unroll
        for (int st = 0; st < KS; ++st) get(st, kept[st]);
    }
    if constexpr (AHEAD) fetch(t, 0);
    for (; t < tend; ++t) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[rb][b] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int cb = 0; cb < cin; cb += C0) {
            if constexpr (!AHEAD) fetch(t, cb);
            __syncthreads();             // the fragments of the chunk before are read
            commit();
            __syncthreads();
            if constexpr (AHEAD) {
                if (cb + C0 < cin) fetch(t, cb + C0);
                else if (t + 1 < tend) fetch(t + 1, 0);
            }
            if constexpr (C0 == 32) {
                if constexpr (!AHEAD) {                // whole chunks alone
                    chunk32_taps(cb);
                } else {
                    const int cc = min(C0, cin - cb);
                    const std::integral_constant<int, 16> c16;
                    if (cc == 32) chunk32(cb);
                    else chunk_small(c16, cb, from_memory(c16, cb));    // the rest of 48 channels
                }
            } else {
                const std::integral_constant<int, C0> c0;
                if constexpr (KEEP) {
                    chunk_small(c0, cb, [&](int st, bf16x8 *w) {
#pragma unroll
                        for (int b = 0; b < NB; ++b) w[b] = kept[st][b];
                    });
                } else {
                    chunk_small(c0, cb, from_memory(c0, cb));
                }
            }
        }
        // lane: output voxel r16 of a row, channels 4 g .. 4 g + 3 of a block
        int X0, Y0, Z0;
        origin(t, X0, Y0, Z0);
        const int i = X0 + r16, k = Z0 + wave;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int co = co0 + b * 16 + 4 * g;
            float bb[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) bb[r] = bias ? bias[co + r] : 0.f;
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const int j = Y0 + rb;
                if (i >= n || j >= n || k >= n) continue;
                bf16x4 o;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float val = acc[rb][b][r] + bb[r];
                    if (relu) val = val > 0.f ? val : 0.f;
                    o[r] = (__bf16)val;
                }
                *reinterpret_cast<bf16x4 *>(y.p + (size_t)(i + n * (j + n * k)) * y.cs + co) = o;
            }
        }
    }
}

struct ConvTiles {
    int tx, ty, tiles;
    explicit ConvTiles(int n) : tx((n + kTileX - 1) / kTileX), ty((n + kTileY - 1) / kTileY)
    {
        tiles = tx * ty * ((n + kTileZ - 1) / kTileZ);
    }
    // tiles a workgroup of NB blocks takes in turn, where fit of them are on the chip at once
    int run(int groups, int fit) const { return (tiles * groups + fit - 1) / fit; }
};

template <int NB, int C0, bool AHEAD>
static void conv_lds_launch(const ConvTiles &t, int per, Tensor x, int cin, const __bf16 *wt, int kpad, int cout,
                            const float *bias, Tensor y, int relu, hipStream_t s)
{
    const dim3 grid((unsigned)((t.tiles + per - 1) / per), (unsigned)(cout / (16 * NB)));
    hipLaunchKernelGGL((conv3d_fwd_lds_k<NB, C0, AHEAD>), grid, dim3(256), 0, s, x, cin, wt, kpad, bias, y, relu, t.tx, t.ty,
                       t.tiles, per);
}

// Whole chunks of 32 input channels: as many blocks of output channels share a staged
// tile as leave 1.5 workgroups per CU (64 -> 64 at 33^3 with NB = 1, 2 and 4 43, 33
// and 35 us, 49^3 98, 89 and 85, 97^3 563, 522 and 489; 32 -> 32 at 41^3 12.8 and 13.9 with NB
// = 1 and 2, 49^3 21 and 18.7).
static void conv_lds32(Tensor x, int cin, const __bf16 *wt, int kpad, int cout, const float *bias, Tensor y, int relu,
                       hipStream_t s)
{
    const ConvTiles t(y.n);
    const int nb = cout / 16, want = 384;
    auto shared = [&](int k) { return nb % k == 0 && t.tiles * (nb / k) >= want; };
    if (shared(4)) conv_lds_launch<4, 32, false>(t, 1, x, cin, wt, kpad, cout, bias, y, relu, s);
    else if (shared(3)) conv_lds_launch<3, 32, false>(t, 1, x, cin, wt, kpad, cout, bias, y, relu, s);
    else if (shared(2)) conv_lds_launch<2, 32, false>(t, 1, x, cin, wt, kpad, cout, bias, y, relu, s);
    else conv_lds_launch<1, 32, false>(t, 1, x, cin, wt, kpad, cout, bias, y, relu, s);
}

// 48 input channels.  A workgroup's run of tiles costs its length times 4, 5, 7 or 9 for
// NB = 1 to 4 (768 workgroups of the first fit the CUs, 512 of the others), so the
// shortest is taken: 48 -> 48 channels at 49^3 47 us with NB = 1, 53 with 3, at 97^3 285 against
// 226; 48 -> 64 at 33^3 26, 21 and 24 with NB = 1, 2 and 4, at 97^3 408, 330 and 306.
static void conv_lds48(Tensor x, int cin, const __bf16 *wt, int kpad, int cout, const float *bias, Tensor y, int relu,
                       hipStream_t s)
{
    const ConvTiles t(y.n);
    const int nb = cout / 16, weight[5] = {0, 4, 5, 7, 9};
    int best = 1, per[5] = {0, t.run(nb, 768)};
    for (int k = 2; k <= 4; ++k) {
        if (nb % k) continue;
        per[k] = t.run(nb / k, 512);
        if (per[k] * weight[k] < per[best] * weight[best]) best = k;
    }
    switch (best) {
    case 2: conv_lds_launch<2, 32, true>(t, per[2], x, cin, wt, kpad, cout, bias, y, relu, s); break;
    case 3: conv_lds_launch<3, 32, true>(t, per[3], x, cin, wt, kpad, cout, bias, y, relu, s); break;
    case 4: conv_lds_launch<4, 32, true>(t, per[4], x, cin, wt, kpad, cout, bias, y, relu, s); break;
    default: conv_lds_launch<1, 32, true>(t, per[1], x, cin, wt, kpad, cout, bias, y, relu, s);
    }
}

template <int NB>
static void conv_lds(Tensor x, int cin, const __bf16 *wt, int kpad, int cout, const float *bias, Tensor y, int relu,
                     hipStream_t s)
{
    // as many workgroups as fit the CUs' LDS (31.1 and 10.4 KB), each with a run of tiles whose loads it overlaps
    const ConvTiles t(y.n);
    const int per = t.run(cout / (16 * NB), cin == 16 ? 1280 : 1536);
    if (cin == 16) conv_lds_launch<NB, 16, true>(t, per, x, cin, wt, kpad, cout, bias, y, relu, s);
    else conv_lds_launch<NB, 8, true>(t, per, x, cin, wt, kpad, cout, bias, y, relu, s);
}

template <int NB>
static void conv_fwd_nb(Tensor x, int cin, const __bf16 *wt, int kpad, const float *bias, Tensor y, int stride,
                        int relu, hipStream_t s)
{
    const int Nout = y.n * y.n * y.n;
    // 96 and 128 output channels keep the order of conv3d_fwd_k, all channels of a tap before the next tap, which
    // the tile kernel follows up to 32 input channels
    if (stride == 1 && (cin == 8 || cin == 16 || cin == 32 || (NB <= 4 && (cin % 32 == 0 || cin == 48)))) {
        if (cin >= 32) {
            if (cin == 48) conv_lds48(x, cin, wt, kpad, 16 * NB, bias, y, relu, s);
            else conv_lds32(x, cin, wt, kpad, 16 * NB, bias, y, relu, s);
            return;
        }
        // With 16 and 8 input channels up to three blocks share a staged tile where that leaves two workgroups per CU.
        const int blocks = ConvTiles(y.n).tiles, want = 512;
        if (NB % 3 == 0 && blocks * (NB / 3) >= want) conv_lds<3>(x, cin, wt, kpad, 16 * NB, bias, y, relu, s);
        else if (NB % 2 == 0 && blocks * (NB / 2) >= want) conv_lds<2>(x, cin, wt, kpad, 16 * NB, bias, y, relu, s);
        else conv_lds<1>(x, cin, wt, kpad, 16 * NB, bias, y, relu, s);
        return;
    }
    // RB row blocks per wave while the grid keeps at least ~1024 workgroups
    if (Nout >= 1024 * 256 && NB <= 4) {
        hipLaunchKernelGGL((conv3d_fwd_k<NB, 4>), dim3((Nout + 255) / 256), dim3(256), 0, s, x, cin, wt, kpad, bias, y,
                           stride, relu);
    } else if (Nout >= 1024 * 128) {
        hipLaunchKernelGGL((conv3d_fwd_k<NB, 2>), dim3((Nout + 127) / 128), dim3(256), 0, s, x, cin, wt, kpad, bias, y,
                           stride, relu);
    } else {
        hipLaunchKernelGGL((conv3d_fwd_k<NB, 1>), dim3((Nout + 63) / 64), dim3(256), 0, s, x, cin, wt, kpad, bias, y,
                           stride, relu);
    }
}

void launch_conv3d_fwd(Tensor x, int cin, const __bf16 *wt, int kpad, int cout, const float *bias, Tensor y,
                       int stride, int relu, hipStream_t s)
{
    switch (cout / 16) {
    case 1: conv_fwd_nb<1>(x, cin, wt, kpad, bias, y, stride, relu, s); break;
    case 2: conv_fwd_nb<2>(x, cin, wt, kpad, bias, y, stride, relu, s); break;
    case 3: conv_fwd_nb<3>(x, cin, wt, kpad, bias, y, stride, relu, s); break;
    case 4: conv_fwd_nb<4>(x, cin, wt, kpad, bias, y, stride, relu, s); break;
    case 6: conv_fwd_nb<6>(x, cin, wt, kpad, bias, y, stride, relu, s); break;
    case 8: conv_fwd_nb<8>(x, cin, wt, kpad, bias, y, stride, relu, s); break;
    default: break;   // rejected by the caller
    }
}

// Weights for the input gradient: W'[ci, tap' cout + co] = W[co, tap cin + ci],
// tap' = 26 - tap (the mirrored offset), so dx = conv(dy, W') with stride 1.
__global__ void dgrad_weights_k(const __bf16 *__restrict__ wt, int cin, int cout, int kpad, __bf16 *__restrict__ wd,
                                int kpad_d)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= cin * kpad_d) return;
    const int ci = t / kpad_d, kk = t - ci * kpad_d;
    __bf16 v = (__bf16)0.f;
    if (kk < 27 * cout) {
        const int tapd = kk / cout, co = kk - tapd * cout;
        v = wt[(size_t)co * kpad + (26 - tapd) * cin + ci];
    }
    wd[t] = v;
}

void launch_dgrad_weights(const __bf16 *wt, int cin, int cout, int kpad, __bf16 *wd, int kpad_d, hipStream_t s)
{
    const int cnt = cin * kpad_d;
    hipLaunchKernelGGL(dgrad_weights_k, dim3((cnt + 255) / 256), dim3(256), 0, s, wt, cin, cout, kpad, wd, kpad_d);
}

// Zero-insertion of a stride-2 output gradient onto the input grid; one
// thread per (voxel, group of 8 channels), 16-byte accesses.
__global__ void dilate_k(Tensor src, Tensor dst, int c)
{
    const int g8 = c / 8;
    const size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    const int nf = dst.n;
    const size_t N = (size_t)nf * nf * nf;
    if (t >= N * g8) return;
    const int v = (int)(t / g8), grp = (int)(t - (size_t)v * g8);
    int i, j, k;
    decode3(v, nf, i, j, k);
    const bool even = !((i | j | k) & 1);
    const int nc = src.n;
    bf16x8 val = {};
    if (even) {
        const size_t vc = (size_t)((i >> 1) + nc * ((j >> 1) + nc * (k >> 1)));
        val = *reinterpret_cast<const bf16x8 *>(src.p + vc * src.cs + 8 * grp);
    }
    *reinterpret_cast<bf16x8 *>(dst.p + (size_t)v * dst.cs + 8 * grp) = val;
}

void launch_dilate(Tensor src, Tensor dst, int c, hipStream_t s)
{
    const size_t cnt = (size_t)dst.n * dst.n * dst.n * (c / 8);
    hipLaunchKernelGGL(dilate_k, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, s, src, dst, c);
}

// Weight gradient: partial[split, co, kk] = sum over the split's output voxels
// o of dy[o, co] X[o, kk], X[o, tap cin + ci] = x[s o + d(tap), ci].  Rows = co,
// columns = kk, K = voxels, 32 consecutive o per MFMA from the split's start,
// so every column is one chain of MFMAs whichever columns share a tile.
//
// Channel-last tensors have K as their slow axis, so the operands are
// transposed on their way through LDS.  A workgroup takes one split, 16 input
// channels, 16 NBW output channels and one dz; wave w owns the three taps of
// row shift (dy, dz) = (w - 1, dz).  It stages its own shifted row of x as
// [channel][voxel] in a ring of three chunks of C voxels; in linear voxel order
// the taps of one (dy, dz) are the same row displaced by one voxel, so one
// 16-byte LDS read and the two dwords beside it give all three fragments.  Rows
// outside the grid are staged as zeros, row ends are masked (mask rows staged
// beside dy).  With stride 2 the even and the odd x of the row are two rows of
// their own and the fragment of tap dx = -1 is the odd row displaced by one; the
// odd row ends in a zero, so no masks are needed.  What bounds it is the latency
// of a wave's global loads and the address and packing work per chunk (the
// fixed splits leave 1300 to 2600 waves for the chip), hence 16-byte loads
// issued DEPTH chunks ahead into register sets of their own and small
// workgroups that spread over all CUs.
//
// The form before this one (wgrad_gather_k) gathered every fragment from global
// memory with 2-byte loads, 16 of them and 8 index divisions per MFMA; it
// serves pointers that are not aligned to 16 bytes.  Measured, same sums bit for
// bit: 48 -> 16 channels at 129^3 5217 -> 540 us, 96 -> 32 at 65^3 1144 ->
// 284 us, 32 -> 32 at 65^3 882 -> 95 us, 128 -> 64 at 33^3 1046 -> 114 us; the
// eleven layers of a 129^3 training step 14.9 -> 1.6 ms.  With one 9-wave
// workgroup per split and channel group and loads one chunk ahead they took
// 2.2 ms (147 workgroups for 256 CUs in the first of these layers).
template <int NBW, int STRIDE>
__global__ void __launch_bounds__(192)
wgrad_rows_k(Tensor x, int cin, Tensor dy, int cout, int kpad, int per_split, float *__restrict__ partial)
{
    static_assert(NBW <= 3, "wave w stages the output channels 16 w .. 16 w + 15");
    constexpr int DEPTH = 3;
    constexpr int C = STRIDE == 1 ? 64 : 32;     // voxels per chunk
    constexpr int RING = 3 * C, PITCH = RING + 8;   // bf16 per staged row: rows 16-byte aligned, halves 32 banks apart
    constexpr int NX = STRIDE;                   // staged rows per channel (stride 2: even and odd x)
    __shared__ __attribute__((aligned(16))) __bf16 xs[3][NX][16][PITCH];
    __shared__ __attribute__((aligned(16))) __bf16 ys[NBW * 16][PITCH];
    __shared__ __attribute__((aligned(16))) unsigned msk[2][RING / 2];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int g = lane >> 4, r16 = lane & 15;
    const int nout = dy.n, nin = x.n, Nout = nout * nout * nout;
    const int dz = blockIdx.z % 3;
    const int split = blockIdx.x, c0 = blockIdx.y * 16, co0 = (blockIdx.z / 3) * 16 * NBW;
    const int sy = w - 1, sz = dz - 1;
    const int ob = split * per_split, oe = min(Nout, ob + per_split);

    // Staging: this lane's voxel pair of a chunk and its 8 channels (half);
    // with stride 2 also the row it stages (even or odd x).
    const int pair = STRIDE == 1 ? (lane & 31) : (lane & 15);
    const int half = STRIDE == 1 ? (lane >> 5) : ((lane >> 4) & 1);
    const int odd = STRIDE == 1 ? 0 : (lane >> 5);
    const bool chan_ok = c0 + 8 * half < cin;
    int o = ob + 2 * pair, i, j, k;              // the pair's first voxel of the next chunk to load
    decode3(o, nout, i, j, k);
    const int di = C % nout, dj = C / nout % nout, dk = C / nout / nout;   // one chunk further
    const __bf16 *xp = x.p + (chan_ok ? c0 + 8 * half : c0);
    const bool stage_y = w < NBW && (STRIDE == 1 || lane < 32);
    const __bf16 *yp = dy.p + (stage_y ? co0 + 16 * w + 8 * half : co0);
    struct Set {
        bf16x8 x[2], y[2];
        unsigned m, okx, oky;
    };
    // Every lane loads from an address clamped into the tensors and masks what it stores: a load in a
    // branch, or a value masked at once, would be waited for where it is issued.
    auto load = [&](Set &r) {
        int a = i, b = j, c = k;
        r.m = r.okx = r.oky = 0;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int oo = o + e;
            const int xi = STRIDE * a + odd, xj = STRIDE * b + sy, xk = STRIDE * c + sz;
            const int ci = min(xi, nin - 1), cj = min(max(xj, 0), nin - 1), ck = min(max(xk, 0), nin - 1);
            r.x[e] = *reinterpret_cast<const bf16x8 *>(xp + (size_t)(ci + nin * (cj + nin * ck)) * x.cs);
            r.y[e] = *reinterpret_cast<const bf16x8 *>(yp + (size_t)(stage_y ? min(oo, Nout - 1) : 0) * dy.cs);
            const unsigned h = e ? 0xffff0000u : 0xffffu;
            if (chan_ok && oo < Nout && xi == ci && xj == cj && xk == ck) r.okx |= h;
            if (oo < oe) r.oky |= h;
            if (oo < oe && a != (half ? nout - 1 : 0)) r.m |= h;
            ++a;
            const int wa = a == nout;
            a = wa ? 0 : a;
            b += wa;
            const int wb = b == nout;
            b = wb ? 0 : b;
            c += wb;
        }
        o += C;
        i += di;
        const int wi = i >= nout;
        i -= wi ? nout : 0;
        j += dj + wi;
        const int wj = j >= nout;
        j -= wj ? nout : 0;
        k += dk + wj;
    };
    auto store = [&](const Set &r, int slot) {
        const int p = slot * C + 2 * pair;
        union U {
            bf16x8 v;
            unsigned short h[8];
        };
        U a, b;
        a.v = r.x[0];
        b.v = r.x[1];
#pragma unroll
        for (int q = 0; q < 8; ++q)
            *reinterpret_cast<unsigned *>(&xs[w][odd][8 * half + q][p]) =
                ((unsigned)a.h[q] | ((unsigned)b.h[q] << 16)) & r.okx;
        if (stage_y) {
            a.v = r.y[0];
            b.v = r.y[1];
#pragma unroll
            for (int q = 0; q < 8; ++q)
                *reinterpret_cast<unsigned *>(&ys[16 * w + 8 * half + q][p]) =
                    ((unsigned)a.h[q] | ((unsigned)b.h[q] << 16)) & r.oky;
        }
        if (STRIDE == 1 && w == 2) msk[half][p >> 1] = r.m;
    };

    f32x4 acc[3][NBW];
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int b = 0; b < NBW; ++b) acc[d][b] = f32x4{0.f, 0.f, 0.f, 0.f};

    // The last slot is read as the voxels before the split's first one (tap
    // dx = -1 of voxel ob): the last voxel of the split before, from the same row.
    if (lane < 16 * NX) {
        __bf16 v = (__bf16)0.f;
        const int ch = lane & 15, row = lane >> 4;
        if (ob > 0) {
            int pi, pj, pk;
            decode3(ob - 1, nout, pi, pj, pk);
            const int xi = STRIDE * pi + row, xj = STRIDE * pj + sy, xk = STRIDE * pk + sz;
            if (c0 + ch < cin && xi < nin && xj >= 0 && xj < nin && xk >= 0 && xk < nin)
                v = x.p[(size_t)(xi + nin * (xj + nin * xk)) * x.cs + c0 + ch];
        }
        xs[w][row][ch][RING - 2] = (__bf16)0.f;
        xs[w][row][ch][RING - 1] = v;
    }

    // chunk c from its slot: MFMAs of 32 voxels each
    auto compute = [&](int c, int slot) {
#pragma unroll
        for (int st = 0; st < C / 32; ++st) {
            if (ob + c * C + 32 * st >= oe) break;
            const int p = slot * C + 32 * st + 8 * g;
            bf16x8 a[NBW];
#pragma unroll
            for (int b = 0; b < NBW; ++b) a[b] = *reinterpret_cast<const bf16x8 *>(&ys[16 * b + r16][p]);
            union F {
                bf16x8 v;
                unsigned d[4];
            };
            F f0, f1, f2, m;
            const __bf16 *row = xs[w][NX - 1][r16];
            m.v = *reinterpret_cast<const bf16x8 *>(row + p);
            const unsigned before = *reinterpret_cast<const unsigned *>(row + (p == 0 ? RING - 2 : p - 2));
            f0.d[0] = __builtin_amdgcn_alignbit(m.d[0], before, 16);
            f0.d[1] = __builtin_amdgcn_alignbit(m.d[1], m.d[0], 16);
            f0.d[2] = __builtin_amdgcn_alignbit(m.d[2], m.d[1], 16);
            f0.d[3] = __builtin_amdgcn_alignbit(m.d[3], m.d[2], 16);
            if constexpr (STRIDE == 1) {
                const unsigned after = *reinterpret_cast<const unsigned *>(row + (p + 8 == RING ? 0 : p + 8));
                f1.v = m.v;
                f2.d[0] = f0.d[1];
                f2.d[1] = f0.d[2];
                f2.d[2] = f0.d[3];
                f2.d[3] = __builtin_amdgcn_alignbit(after, m.d[3], 16);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    f0.d[q] &= msk[0][(p >> 1) + q];
                    f2.d[q] &= msk[1][(p >> 1) + q];
                }
            } else {
                f1.v = *reinterpret_cast<const bf16x8 *>(&xs[w][0][r16][p]);
                f2.v = m.v;
            }
#pragma unroll
            for (int b = 0; b < NBW; ++b) {
                acc[0][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[b], f0.v, acc[0][b], 0, 0, 0);
                acc[1][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[b], f1.v, acc[1][b], 0, 0, 0);
                acc[2][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[b], f2.v, acc[2][b], 0, 0, 0);
            }
        }
    };

    // Step c stores chunk c + 1, asks for chunk c + 1 + DEPTH and works on chunk
    // c.  dy and the masks of chunk c were stored by their waves before the
    // barrier of step c; a wave past it stores chunk c + 2, whose slot held
    // chunk c - 1, which no wave reads any more.
    Set r[DEPTH];
    load(r[0]);
    store(r[0], 0);
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) load(r[d]);
    const int nchunk = (oe - ob + C - 1) / C;
    for (int c = 0; c < nchunk; c += DEPTH) {     // slot of chunk c: c mod 3, and DEPTH = 3
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {     // past the last chunk: nothing to compute, clamped loads
            store(r[d], (d + 1) % 3);
            load(r[d]);
            __syncthreads();
            compute(c + d, d);
        }
    }
    if (c0 + r16 >= cin) return;
    float *P = partial + (size_t)split * cout * kpad;
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int b = 0; b < NBW; ++b)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4)
                P[(size_t)(co0 + 16 * b + 4 * g + r4) * kpad + (3 * (w + 3 * dz) + d) * cin + c0 + r16] = acc[d][b][r4];
}

// The same sums with every fragment gathered by 2-byte loads, one wave per
// (16 co x 16 kk) tile and split: takes pointers of any alignment.
__global__ void __launch_bounds__(256)
wgrad_gather_k(Tensor x, int cin, Tensor dy, int cout, int kpad, int stride, int nsplit, int per_split,
        float *__restrict__ partial)
{
    const int lane = threadIdx.x & 63;
    const int gw = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int nct = cout / 16, nkt = kpad / 16;
    const int ntile = nct * nkt;
    if (gw >= ntile * nsplit) return;
    const int split = gw / ntile, tile = gw - split * ntile;
    const int ct = tile / nkt, kt = tile - ct * nkt;
    const int g = lane >> 4, r16 = lane & 15;
    const int co = ct * 16 + r16, kk = kt * 16 + r16;
    const int nout = dy.n, nin = x.n, Nout = nout * nout * nout;
    const bool kvalid = kk < 27 * cin;
    const int tap = kvalid ? kk / cin : 0, ci = kvalid ? kk - tap * cin : 0;
    const int dxo = tap % 3 - 1, dyo = (tap / 3) % 3 - 1, dzo = tap / 9 - 1;
    const int ob = split * per_split, oe = min(Nout, ob + per_split);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int o0 = ob; o0 < oe; o0 += 32) {
        bf16x8 a, b;
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) {
            const int o = o0 + 8 * g + jj;
            __bf16 av = (__bf16)0.f, bv = (__bf16)0.f;
            if (o < oe) {
                av = dy.p[(size_t)o * dy.cs + co];
                if (kvalid) {
                    int i, j, k;
                    decode3(o, nout, i, j, k);
                    i = stride * i + dxo;
                    j = stride * j + dyo;
                    k = stride * k + dzo;
                    if (i >= 0 && i < nin && j >= 0 && j < nin && k >= 0 && k < nin)
                        bv = x.p[(size_t)(i + nin * (j + nin * k)) * x.cs + ci];
                }
            }
            a[jj] = av;
            b[jj] = bv;
        }
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
    }
    float *P = partial + (size_t)split * cout * kpad;
#pragma unroll
    for (int r = 0; r < 4; ++r) P[(size_t)(ct * 16 + 4 * g + r) * kpad + kk] = acc[r];
}

// out[t] = sum_s partial[s, t] in fixed order, 0 in the padding of a weight
// row (t % kpad >= kreal); 16 loads in flight per thread, added in order.
__global__ void split_reduce_k(const float *__restrict__ partial, int nsplit, int count, int kpad, int kreal,
                               float *__restrict__ out)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= count) return;
    float s = 0.f;
    if (t % kpad < kreal) {
        int q = 0;
        for (; q + 16 <= nsplit; q += 16) {
            float v[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) v[e] = partial[(size_t)(q + e) * count + t];
#pragma unroll
            for (int e = 0; e < 16; ++e) s += v[e];
        }
        for (; q < nsplit; ++q) s += partial[(size_t)q * count + t];
    }
    out[t] = s;
}

int wgrad_splits(int cout, int kpad, int nout)
{
    const int ntile = (cout / 16) * (kpad / 16);
    const int Nout = nout * nout * nout;
    int ns = 4096 / ntile;
    if (ns < 1) ns = 1;
    const int maxs = (Nout + 1023) / 1024;
    if (ns > maxs) ns = maxs;
    if (ns > kMaxSplit) ns = kMaxSplit;
    return ns;
}

template <int STRIDE>
static void wgrad_rows(Tensor x, int cin, Tensor dy, int cout, int kpad, int nsplit, int per, float *partial, hipStream_t s)
{
    const unsigned cg = (unsigned)((cin + 15) / 16);
    const int nct = cout / 16;
    // two tiles of output channels share the staged x while 3 waves are left for every CU
    const bool two = nct % 2 == 0 && nsplit * (int)cg * 3 * (nct / 2) >= 256;
    const dim3 grid((unsigned)nsplit, cg, (unsigned)(3 * (two ? nct / 2 : nct)));
    if (two)
        hipLaunchKernelGGL((wgrad_rows_k<2, STRIDE>), grid, dim3(192), 0, s, x, cin, dy, cout, kpad, per, partial);
    else
        hipLaunchKernelGGL((wgrad_rows_k<1, STRIDE>), grid, dim3(192), 0, s, x, cin, dy, cout, kpad, per, partial);
}

void launch_wgrad(Tensor x, int cin, Tensor dy, int cout, int kpad, int stride, float *partial, float *dw, hipStream_t s)
{
    const int nsplit = wgrad_splits(cout, kpad, dy.n);
    const int Nout = dy.n * dy.n * dy.n;
    int per = (Nout + nsplit - 1) / nsplit;
    per = (per + 31) / 32 * 32;
    // slot widths are multiples of 8 channels, so an aligned base aligns every 8-channel load
    const bool aligned = (((uintptr_t)x.p | (uintptr_t)dy.p) & 15) == 0 && x.cs % 8 == 0 && dy.cs % 8 == 0;
    if (aligned && stride == 1) {
        wgrad_rows<1>(x, cin, dy, cout, kpad, nsplit, per, partial, s);
    } else if (aligned) {
        wgrad_rows<2>(x, cin, dy, cout, kpad, nsplit, per, partial, s);
    } else {
        const int waves = (cout / 16) * (kpad / 16) * nsplit;
        hipLaunchKernelGGL(wgrad_gather_k, dim3((waves + 3) / 4), dim3(256), 0, s, x, cin, dy, cout, kpad, stride, nsplit,
                           per, partial);
    }
    const int cnt = cout * kpad;
    hipLaunchKernelGGL(split_reduce_k, dim3((cnt + 255) / 256), dim3(256), 0, s, partial, nsplit, cnt, kpad, 27 * cin, dw);
}

// Splits of a voxel range for the fixed-order reductions below: at most
// kMaxSplit workgroups, each over a contiguous range.
static int reduce_splits(int N)
{
    int ns = (N + 2047) / 2048;
    return ns < 1 ? 1 : (ns > kMaxSplit ? kMaxSplit : ns);
}

// The gradient before the ReLU of a layer, in place, and its bias gradient:
// g[v, c] += add[v, c] (rounded once to BF16; add.p null: nothing), 0 where the
// ReLU output y[v, c] is 0, partial[split, c] = sum over the split's voxels of g.
// Workgroup = split; a thread takes two channels of voxels l + q (256 / c), l
// its place among 256 / c voxels (c divides 256), so that a channel's sum is one
// chain per l, combined in a fixed order at the end.  The chain and its few
// splits leave little parallelism: UN steps of a chain are loaded at once.  One
// pass for what were up to three, whose sums waited for every load: 16 channels
// at 129^3 89 (add) + 84 (ReLU) + 126 (sums) -> 120 us.
template <bool ADD>
__global__ void __launch_bounds__(128) pre_grad_k(Tensor g, Tensor add, Tensor y, int c, int per, float *__restrict__ partial)
{
    constexpr int UN = 16;
    __shared__ float sh[256];
    const int N = g.n * g.n * g.n;
    const int vb = blockIdx.x * per, ve = min(N, vb + per);
    const int hc = c / 2, ch = 2 * ((int)threadIdx.x % hc), lanes = 256 / c, l = threadIdx.x / hc;
    float s0 = 0.f, s1 = 0.f;
    for (int v0 = vb + l; v0 < ve; v0 += UN * lanes) {
        bf16x2 gv[UN], av[UN], yv[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const size_t v = (size_t)min(v0 + u * lanes, ve - 1);
            gv[u] = *reinterpret_cast<const bf16x2 *>(g.p + v * g.cs + ch);
            yv[u] = *reinterpret_cast<const bf16x2 *>(y.p + v * y.cs + ch);
            if (ADD) av[u] = *reinterpret_cast<const bf16x2 *>(add.p + v * add.cs + ch);
        }
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            if (v0 + u * lanes >= ve) break;
            bf16x2 r = gv[u];
            if (ADD) {
                r[0] = (__bf16)((float)r[0] + (float)av[u][0]);
                r[1] = (__bf16)((float)r[1] + (float)av[u][1]);
            }
            if (!((float)yv[u][0] > 0.f)) r[0] = (__bf16)0.f;
            if (!((float)yv[u][1] > 0.f)) r[1] = (__bf16)0.f;
            *reinterpret_cast<bf16x2 *>(g.p + (size_t)(v0 + u * lanes) * g.cs + ch) = r;
            s0 += (float)r[0];
            s1 += (float)r[1];
        }
    }
    sh[l * c + ch] = s0;
    sh[l * c + ch + 1] = s1;
    __syncthreads();
    if ((int)threadIdx.x < c) {
        float t = 0.f;
        for (int q = 0; q < lanes; ++q) t += sh[q * c + threadIdx.x];
        partial[(size_t)blockIdx.x * c + threadIdx.x] = t;
    }
}

void launch_pre_grad(Tensor g, Tensor add, Tensor y, int c, float *partial, float *db, hipStream_t s)
{
    const int N = g.n * g.n * g.n;
    const int nsplit = reduce_splits(N);
    const int per = (N + nsplit - 1) / nsplit;
    if (add.p) hipLaunchKernelGGL(pre_grad_k<true>, dim3(nsplit), dim3(128), 0, s, g, add, y, c, per, partial);
    else hipLaunchKernelGGL(pre_grad_k<false>, dim3(nsplit), dim3(128), 0, s, g, add, y, c, per, partial);
    hipLaunchKernelGGL(split_reduce_k, dim3(1), dim3(256), 0, s, partial, nsplit, c, c, c, db);
}

// Trilinear 2x up-sampling of vertex-centred grids (n_fine = 2 n_coarse - 1);
// one thread per (fine voxel, group of 8 channels).
__global__ void upsample_k(Tensor src, Tensor dst, int c)
{
    const int g8 = c / 8;
    const size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    const int nf = dst.n, nc = src.n;
    const size_t N = (size_t)nf * nf * nf;
    if (t >= N * g8) return;
    const int v = (int)(t / g8), grp = (int)(t - (size_t)v * g8);
    int i, j, k;
    decode3(v, nf, i, j, k);
    const int i0 = i >> 1, i1 = (i + 1) >> 1, j0 = j >> 1, j1 = (j + 1) >> 1, k0 = k >> 1, k1 = (k + 1) >> 1;
    const float wi = (i & 1) ? 0.5f : 1.f, wj = (j & 1) ? 0.5f : 1.f, wk = (k & 1) ? 0.5f : 1.f;
    const float wi1 = (i & 1) ? 0.5f : 0.f, wj1 = (j & 1) ? 0.5f : 0.f, wk1 = (k & 1) ? 0.5f : 0.f;
    auto at = [&](int a, int b, int cc) {
        return *reinterpret_cast<const bf16x8 *>(src.p + (size_t)(a + nc * (b + nc * cc)) * src.cs + 8 * grp);
    };
    const bf16x8 a000 = at(i0, j0, k0), a100 = at(i1, j0, k0), a010 = at(i0, j1, k0), a110 = at(i1, j1, k0);
    const bf16x8 a001 = at(i0, j0, k1), a101 = at(i1, j0, k1), a011 = at(i0, j1, k1), a111 = at(i1, j1, k1);
    bf16x8 out;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float x00 = wi * (float)a000[e] + wi1 * (float)a100[e];
        const float x10 = wi * (float)a010[e] + wi1 * (float)a110[e];
        const float x01 = wi * (float)a001[e] + wi1 * (float)a101[e];
        const float x11 = wi * (float)a011[e] + wi1 * (float)a111[e];
        out[e] = (__bf16)(wk * (wj * x00 + wj1 * x10) + wk1 * (wj * x01 + wj1 * x11));
    }
    *reinterpret_cast<bf16x8 *>(dst.p + (size_t)v * dst.cs + 8 * grp) = out;
}

void launch_upsample(Tensor src, Tensor dst, int c, hipStream_t s)
{
    const size_t cnt = (size_t)dst.n * dst.n * dst.n * (c / 8);
    hipLaunchKernelGGL(upsample_k, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, s, src, dst, c);
}

// Adjoint of upsample_k: coarse node I gathers w g(2I + d) over d in {-1,0,1}^3,
// w = product over axes of (1 if d = 0 else 1/2).
// one thread per (coarse voxel, group of 8 channels)
__global__ void upsample_adj_k(Tensor gf, Tensor gc, int c)
{
    const int g8 = c / 8;
    const size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    const int nc = gc.n, nf = gf.n;
    const size_t N = (size_t)nc * nc * nc;
    if (t >= N * g8) return;
    const int v = (int)(t / g8), grp = (int)(t - (size_t)v * g8);
    int I, J, K;
    decode3(v, nc, I, J, K);
    float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int dz = -1; dz <= 1; ++dz) {
        const int k = 2 * K + dz;
        if (k < 0 || k >= nf) continue;
        for (int dy = -1; dy <= 1; ++dy) {
            const int j = 2 * J + dy;
            if (j < 0 || j >= nf) continue;
            for (int dx = -1; dx <= 1; ++dx) {
                const int i = 2 * I + dx;
                if (i < 0 || i >= nf) continue;
                const float w = (dx ? 0.5f : 1.f) * (dy ? 0.5f : 1.f) * (dz ? 0.5f : 1.f);
                const bf16x8 a = *reinterpret_cast<const bf16x8 *>(gf.p + (size_t)(i + nf * (j + nf * k)) * gf.cs + 8 * grp);
#pragma unroll
                for (int e = 0; e < 8; ++e) s[e] += w * (float)a[e];
            }
        }
    }
    bf16x8 out;
#pragma unroll
    for (int e = 0; e < 8; ++e) out[e] = (__bf16)s[e];
    *reinterpret_cast<bf16x8 *>(gc.p + (size_t)v * gc.cs + 8 * grp) = out;
}

void launch_upsample_adj(Tensor gf, Tensor gc, int c, hipStream_t s)
{
    const size_t cnt = (size_t)gc.n * gc.n * gc.n * (c / 8);
    hipLaunchKernelGGL(upsample_adj_k, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, s, gf, gc, c);
}

// ------------------------------------------------------------- head, loss

// yhat[v] = b + sum_c w[c] x[v, c] (c a multiple of 8; 16-byte loads, same order)
__global__ void head_fwd_k(Tensor x, int c, const float *__restrict__ w, const float *__restrict__ b, float *__restrict__ yh)
{
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    const int N = x.n * x.n * x.n;
    if (v >= N) return;
    float s = b[0];
    for (int c8 = 0; c8 < c; c8 += 8) {
        const bf16x8 a = *reinterpret_cast<const bf16x8 *>(x.p + (size_t)v * x.cs + c8);
#pragma unroll
        for (int e = 0; e < 8; ++e) s += w[c8 + e] * (float)a[e];
    }
    yh[v] = s;
}

void launch_head_fwd(Tensor x, int c, const float *w, const float *b, float *yh, hipStream_t s)
{
    const int N = x.n * x.n * x.n;
    hipLaunchKernelGGL(head_fwd_k, dim3((N + 255) / 256), dim3(256), 0, s, x, c, w, b, yh);
}

// Backward of the head and of the ReLU below it in one pass over x (the ReLU's
// output): dx[v, c] = dy[v] w[c] (rounded to BF16), 0 where x[v, c] is 0; partial
// sums per split of dy[v] x[v, c] (c < C), of dy[v] (C) and of dx[v, c] (C + 1 ..
// 2 C, the bias gradient of the layer below).  Chains and order as in
// pre_grad_k.
__global__ void __launch_bounds__(128)
head_bwd_k(const float *__restrict__ dyh, Tensor x, int c, const float *__restrict__ w, Tensor dx, int per,
           float *__restrict__ partial)
{
    constexpr int UN = 16;
    __shared__ float sw[256], sb[256], sd[256];
    const int N = x.n * x.n * x.n;
    const int vb = blockIdx.x * per, ve = min(N, vb + per);
    const int hc = c / 2, ch = 2 * ((int)threadIdx.x % hc), lanes = 256 / c, l = threadIdx.x / hc;
    const float w0 = w[ch], w1 = w[ch + 1];
    float s0 = 0.f, s1 = 0.f, b = 0.f, d0 = 0.f, d1 = 0.f;
    for (int v0 = vb + l; v0 < ve; v0 += UN * lanes) {
        float dv[UN];
        bf16x2 xv[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const size_t v = (size_t)min(v0 + u * lanes, ve - 1);
            dv[u] = dyh[v];
            xv[u] = *reinterpret_cast<const bf16x2 *>(x.p + v * x.cs + ch);
        }
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            if (v0 + u * lanes >= ve) break;
            const float d = dv[u], x0 = (float)xv[u][0], x1 = (float)xv[u][1];
            bf16x2 r;
            r[0] = x0 > 0.f ? (__bf16)(d * w0) : (__bf16)0.f;
            r[1] = x1 > 0.f ? (__bf16)(d * w1) : (__bf16)0.f;
            *reinterpret_cast<bf16x2 *>(dx.p + (size_t)(v0 + u * lanes) * dx.cs + ch) = r;
            s0 += d * x0;
            s1 += d * x1;
            b += d;
            d0 += (float)r[0];
            d1 += (float)r[1];
        }
    }
    sw[l * c + ch] = s0;
    sw[l * c + ch + 1] = s1;
    sb[l * c + ch] = b;
    sd[l * c + ch] = d0;
    sd[l * c + ch + 1] = d1;
    __syncthreads();
    const int t = threadIdx.x, row = 2 * c + 1;
    if (t <= 2 * c) {
        const float *src = t < c ? sw + t : (t == c ? sb : sd + (t - c - 1));   // every voxel once in channel 0's sums
        float v = 0.f;
        for (int q = 0; q < lanes; ++q) v += src[q * c];
        partial[(size_t)blockIdx.x * row + t] = v;
    }
}

// dwb: c weights and the bias of the head, then the c bias gradients of the layer below
void launch_head_bwd(const float *dyh, Tensor x, int c, const float *w, Tensor dx, float *partial, float *dwb,
                     hipStream_t s)
{
    const int N = x.n * x.n * x.n;
    const int nsplit = reduce_splits(N);
    const int per = (N + nsplit - 1) / nsplit, row = 2 * c + 1;
    hipLaunchKernelGGL(head_bwd_k, dim3(nsplit), dim3(128), 0, s, dyh, x, c, w, dx, per, partial);
    hipLaunchKernelGGL(split_reduce_k, dim3(1), dim3(256), 0, s, partial, nsplit, row, row, row, dwb);
}

// Mean squared error over interior nodes; dy = 2 (yhat - t) / N_int there, 0 on
// the boundary.  partial[b] per block, then one block.
__global__ void __launch_bounds__(256)
mse_k(const float *__restrict__ yh, const float *__restrict__ tg, int n, float *__restrict__ dy, double *__restrict__ partial)
{
    __shared__ double sh[256];
    const int N = n * n * n;
    const double nint = (double)(n - 2) * (n - 2) * (n - 2);
    double s = 0.0;
    for (int v = blockIdx.x * 256 + threadIdx.x; v < N; v += gridDim.x * 256) {
        int i, j, k;
        decode3(v, n, i, j, k);
        const bool in = i > 0 && j > 0 && k > 0 && i < n - 1 && j < n - 1 && k < n - 1;
        const float d = in ? yh[v] - tg[v] : 0.f;
        dy[v] = (float)(2.0 * d / nint);
        s += (double)d * d;
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = sh[0] / nint;
}

__global__ void sum_k(const double *__restrict__ partial, int nb, double *__restrict__ out)
{
    __shared__ double sh[kLossBlocks];
    for (int b = threadIdx.x; b < nb; b += 64) sh[b] = partial[b];
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int b = 0; b < nb; ++b) s += sh[b];
        out[0] = s;
    }
}

void launch_mse(const float *yh, const float *tg, int n, float *dy, double *partial, double *loss, hipStream_t s)
{
    hipLaunchKernelGGL(mse_k, dim3(kLossBlocks), dim3(256), 0, s, yh, tg, n, dy, partial);
    hipLaunchKernelGGL(sum_k, dim3(1), dim3(64), 0, s, partial, kLossBlocks, loss);
}

// Adam on FP32 master weights, all arrays of the network in one launch; the
// BF16 copy (if any) is refreshed.
__global__ void adam_k(const AdamArray *__restrict__ arrays, int n, float lr, float b1, float b2, float eps, float c1,
                       float c2)
{
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    for (int a = 0; a < n; ++a) {
        const AdamArray A = arrays[a];
        if (t < A.count) {
            const float gt = A.g[t];
            const float mt = b1 * A.m[t] + (1.f - b1) * gt;
            const float vt = b2 * A.v[t] + (1.f - b2) * gt * gt;
            A.m[t] = mt;
            A.v[t] = vt;
            const float wt = A.w[t] - lr * (mt / c1) / (sqrtf(vt / c2) + eps);
            A.w[t] = wt;
            if (A.wb) A.wb[t] = (__bf16)wt;
            return;
        }
        t -= A.count;
    }
}

void launch_adam(const AdamArray *arrays, int n, int total, float lr, int step, hipStream_t s)
{
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
    hipLaunchKernelGGL(adam_k, dim3((total + 255) / 256), dim3(256), 0, s, arrays, n, lr, b1, b2, eps, c1, c2);
}

__global__ void to_bf16_k(const float *__restrict__ src, __bf16 *__restrict__ dst, int count)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < count) dst[t] = (__bf16)src[t];
}

void launch_to_bf16(const float *src, __bf16 *dst, int count, hipStream_t s)
{
    hipLaunchKernelGGL(to_bf16_k, dim3((count + 255) / 256), dim3(256), 0, s, src, dst, count);
}

// --------------------------------------------------------- inputs, outputs

// Network input: channel 0 = Phi_N / cn, channel 1 = h^2 S / cs, further channels
// of the slot (if any) = 0.
__global__ void prep_input_k(int n, const double *__restrict__ phin, const double *__restrict__ base,
                             const double *__restrict__ S, double inv_cn, double h2_cs, Tensor x)
{
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n * n * n) return;
    __bf16 *p = x.p + (size_t)v * x.cs;
    p[0] = (__bf16)(float)((phin[v] - base[v]) * inv_cn);
    p[1] = (__bf16)(float)(S[v] * h2_cs);
    for (int c = 2; c < x.cs; ++c) p[c] = (__bf16)0.f;
}

// Two-channel compact sample -> the network's 8-channel input slot.
__global__ void expand_input_k(const __bf16 *__restrict__ xc, Tensor x)
{
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= x.n * x.n * x.n) return;
    __bf16 *p = x.p + (size_t)v * x.cs;
    p[0] = xc[2 * (size_t)v];
    p[1] = xc[2 * (size_t)v + 1];
    for (int c = 2; c < x.cs; ++c) p[c] = (__bf16)0.f;
}

void launch_expand_input(const __bf16 *xc, Tensor x, hipStream_t s)
{
    const int N = x.n * x.n * x.n;
    hipLaunchKernelGGL(expand_input_k, dim3((N + 255) / 256), dim3(256), 0, s, xc, x);
}

void launch_prep_input(int n, const double *phin, const double *base, const double *S, double inv_cn, double h2_cs,
                       Tensor x, hipStream_t s)
{
    const int N = n * n * n;
    hipLaunchKernelGGL(prep_input_k, dim3((N + 255) / 256), dim3(256), 0, s, n, phin, base, S, inv_cn, h2_cs, x);
}

// out[v] = a * in[v] + base[v] (FP32 -> FP64)
__global__ void scale_out_k(const float *__restrict__ in, int count, double a, const double *__restrict__ base,
                            double *__restrict__ out)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < count) out[t] = a * (double)in[t] + base[t];
}

void launch_scale_out(const float *in, int count, double a, const double *base, double *out, hipStream_t s)
{
    hipLaunchKernelGGL(scale_out_k, dim3((count + 255) / 256), dim3(256), 0, s, in, count, a, base, out);
}

// out[v] = (float)(a * (in[v] - base[v])) (FP64 -> FP32 target)
__global__ void scale_in_k(const double *__restrict__ in, const double *__restrict__ base, int count, double a,
                           float *__restrict__ out)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < count) out[t] = (float)(a * (in[t] - base[t]));
}

void launch_scale_in(const double *in, const double *base, int count, double a, float *out, hipStream_t s)
{
    hipLaunchKernelGGL(scale_in_k, dim3((count + 255) / 256), dim3(256), 0, s, in, base, count, a, out);
}

}  // namespace qm
