// Learned warm start: a small 3D U-Net in bfloat16 with float32 accumulation,
// built from hand-written MFMA convolution kernels (forward, backward-data,
// backward-weight), an Adam optimiser and the element-wise glue, all on the
// device.  The network maps the density contrast of a periodic S^3 mesh (plus
// the scale factor and |f_R0| as constant channels) to the solution u of the
// field equation on that mesh.  The solver uses it at the N/4 level of an N^3
// problem and prolongs the prediction to the finest level as the initial
// guess of the multigrid solve (Sec. 3.3 step 2 takes the initial guess from
// outside; multigrid still iterates to the same tolerance).
//
// Architecture (channels): 16 -> [16,16] -> pool -> [32,32] -> pool -> [64,64]
// -> up, concat(64+32) -> [32,32] -> up, concat(32+16) -> [16,16] -> 1x1 -> 1,
// every bracketed entry a 3^3 periodic convolution with bias and ReLU; pool is
// the 2^3 mean, up the 2^3 nearest-neighbour copy.  Activations are
// channels-last ([voxel][channel], voxel = ((b S + z) S + y) S + x).
//
// Convolution as an implicit GEMM on v_mfma_f32_16x16x32_bf16: rows are
// voxels, columns output channels, and the reduction runs over chunks of the
// input channels staged in LDS with their halo, and within a chunk over the
// 27 taps and its channels in steps of 32 (8 consecutive channels of one tap
// per lane).  The backward-data pass is the same kernel on
// the output gradient with the taps mirrored and the weight matrix transposed;
// the backward-weight pass reduces over voxels, its fragments read from LDS by
// the transpose load.
#include "mgfr_internal.h"
#include "mgfr_ops.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <random>
#include <vector>

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// eight bf16 at an address that need not be a multiple of 16
typedef __bf16 bf16x8_any __attribute__((ext_vector_type(8), aligned(2)));

namespace mgfr {

namespace {

#ifndef MGFR_CONV_WAVES
#define MGFR_CONV_WAVES 4
#endif
#ifndef MGFR_CONV_MT
#define MGFR_CONV_MT 4
#endif
constexpr int kConvWaves = MGFR_CONV_WAVES;  // waves per workgroup in the forward kernel
constexpr int kConvMT = MGFR_CONV_MT;        // 16-voxel row tiles per wave (256 voxels per workgroup)
// LDS stride of a staged voxel: 32-channel chunks get 8 bf16 of padding (the
// 16-byte A-fragment reads of 16 consecutive voxels then spread over the
// banks: 1.4x faster on those layers; 16-channel chunks are faster without)
__host__ __device__ constexpr int conv_stride(int CC) { return CC == 32 ? CC + 8 : CC; }
constexpr float kUScale = 5.0f; // network output = u / kUScale

__device__ __forceinline__ float bf2f(__bf16 x) { return (float)x; }
__device__ __forceinline__ __bf16 f2bf(float x) { return (__bf16)x; }

// -------------------------------------------------------------- convolution

// Y[v][o] = act(sum_{t,c} X[v + off(t)][c] W[t][o][c] + bias[o]) on B periodic S^3
// volumes.  W layout [27][Cout][Cin].  Cin % 8 == 0, Cout % 16 == 0, Cout <= 96, S >= 8.
//
// A workgroup owns a tile of 256 output voxels, TX x 8 x TZ with TX = min(S, 16)
// and TZ = 256 / (8 TX); it stages the tile and a one-voxel periodic halo of
// the input in LDS, CC channels at a time (CC = 32, 16 or 8, dividing Cin),
// so that the 27 taps read the activations from LDS instead of gathering them
// 27 times from global memory.  Each wave computes 4 row tiles of 16 voxels
// against all Cout columns; the weights come from global memory (L2/L1 hits:
// every workgroup reads the same few KB), each k-step's fragments loaded
// while the previous step's MFMAs run.

// NT column tiles of 16 output channels per workgroup, starting at channel
// 16 NT blockIdx.y (a template parameter: the accumulators of the 16-channel
// layers then take 16 registers, not 96; small grids split Cout over
// blockIdx.y to fill the chip)
template <int NT>
__global__ __launch_bounds__(64 * kConvWaves) void k_conv3d(const __bf16 *__restrict__ X, int lgS, int Cin,
                                                             const __bf16 *__restrict__ W,
                                                             const float *__restrict__ bias, int Cout, int relu,
                                                             const __bf16 *__restrict__ M,
                                                             __bf16 *__restrict__ Y, float *__restrict__ Y32)
{
    extern __shared__ __attribute__((aligned(16))) __bf16 sX[];  // [halo voxels][CC], sized at launch
    __shared__ int sTap[32];  // LDS offset (in voxels) of each tap's neighbour
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int S = 1 << lgS, sm = S - 1;
    const int lgX = lgS < 4 ? lgS : 4;
    const int TX = 1 << lgX, TY = 8, TZ = (16 * kConvMT * kConvWaves) / (TX * TY);
    const int HX = TX + 2, HY = TY + 2, HZ = TZ + 2, HV = HX * HY * HZ;
    unsigned bi = blockIdx.x;
    const int ntx = S / TX, nty = S / TY, ntz = S / TZ;
    const int x0 = (int)(bi % ntx) * TX;
    bi /= ntx;
    const int y0 = (int)(bi % nty) * TY;
    bi /= nty;
    const int z0 = (int)(bi % ntz) * TZ;
    const size_t vol = bi / ntz;
    const int g = lane >> 4, r16 = lane & 15;
    const int ocol0 = 16 * NT * (int)blockIdx.y;
    if (threadIdx.x < 32) {
        const int t = threadIdx.x < 27 ? threadIdx.x : 0;
        sTap[threadIdx.x] = ((t / 9 - 1) * HY + ((t / 3) % 3 - 1)) * HX + (t % 3 - 1);
    }
    // halo-tile voxel of each row this lane feeds to the A operand
    int hb[kConvMT];
#pragma unroll
    for (int mt = 0; mt < kConvMT; ++mt) {
        const int lv = 16 * (w * kConvMT + mt) + r16;
        const int lx = lv & (TX - 1), ly = (lv >> lgX) & (TY - 1), lz = lv >> (lgX + 3);
        hb[mt] = ((lz + 1) * HY + (ly + 1)) * HX + (lx + 1);
    }
    f32x4 acc[kConvMT][NT];
#pragma unroll
    for (int mt = 0; mt < kConvMT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int lgC = (Cin % 32 == 0) ? 5 : ((Cin % 16 == 0) ? 4 : 3);  // chunk CC = 2^lgC channels
    const int CC = 1 << lgC;
    const int q8 = CC >> 3, KC = 27 * CC, CS = conv_stride(CC);
    for (int cc0 = 0; cc0 < Cin; cc0 += CC) {
        __syncthreads();  // the previous chunk's readers are done
        for (int idx = threadIdx.x; idx < HV * q8; idx += 64 * kConvWaves) {
            const int hv = idx / q8, q = idx - hv * q8;
            const int hx = hv % HX, t = hv / HX, hy = t % HY, hz = t / HY;
            const size_t src = ((((vol << lgS) + (size_t)((z0 + hz - 1) & sm)) << (2 * lgS)) +
                                ((size_t)((y0 + hy - 1) & sm) << lgS) + (size_t)((x0 + hx - 1) & sm));
            *(bf16x8 *)(sX + hv * CS + 8 * q) = *(const bf16x8 *)(X + src * Cin + cc0 + 8 * q);
        }
        __syncthreads();
        // weight fragments from global memory, loaded one k-step ahead
        auto loadB = [&](int k0, bf16x8 *b) {
            const int kk = k0 + 8 * g;
            const bool valid = kk < KC;
            const int tap = valid ? kk >> lgC : 0;
            const int c = valid ? kk & (CC - 1) : 0;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                b[nt] = valid ? *(const bf16x8 *)(W + ((size_t)tap * Cout + ocol0 + 16 * nt + r16) * Cin + cc0 + c)
                              : bf16x8{};
        };
        bf16x8 bcur[NT], bnxt[NT] = {};
        loadB(0, bcur);
        for (int k0 = 0; k0 < KC; k0 += 32) {
            if (k0 + 32 < KC) loadB(k0 + 32, bnxt);
            const int kk = k0 + 8 * g;
            const bool valid = kk < KC;
            const int tap = valid ? kk >> lgC : 0;
            const int c = valid ? kk & (CC - 1) : 0;
            const int toff = sTap[tap];
            bf16x8 a[kConvMT];
#pragma unroll
            for (int mt = 0; mt < kConvMT; ++mt)
                a[mt] = valid ? *(const bf16x8 *)(sX + (hb[mt] + toff) * CS + c) : bf16x8{};
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int mt = 0; mt < kConvMT; ++mt)
                    acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[mt], bcur[nt], acc[mt][nt], 0, 0, 0);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) bcur[nt] = bnxt[nt];
        }
    }
#pragma unroll
    for (int mt = 0; mt < kConvMT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            {
                const int o = ocol0 + 16 * nt + r16;
                const float bo = bias ? bias[o] : 0.f;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int lv = 16 * (w * kConvMT + mt) + 4 * g + j;
                    const int lx = lv & (TX - 1), ly = (lv >> lgX) & (TY - 1), lz = lv >> (lgX + 3);
                    const size_t v = ((((vol << lgS) + (size_t)(z0 + lz)) << lgS) + (size_t)(y0 + ly)) * (size_t)S +
                                      (size_t)(x0 + lx);
                    float val = acc[mt][nt][j] + bo;
                    if (relu) val = fmaxf(val, 0.f);
                    if (M && !(bf2f(M[v * Cout + o]) > 0.f)) val = 0.f;
                    if (Y) Y[v * Cout + o] = f2bf(val);
                    if (Y32) Y32[v * Cout + o] = val;
                }
            }
        }
}

// Input of a layer: C channels per voxel of x or, with a skip connection, the
// nearest-neighbour upsampling of x (C channels per voxel of the mesh of half the
// side) followed by the Cs channels of skip.  A chunk of channels comes from one
// of the two (C is a multiple of it), so that no concatenated copy is written
// (62 us of the 556 us of a 128^3 prediction, and the copies were read from HBM:
// 48 -> 16 channels 145 -> 124 us then, its weight gradient 213 -> 165 us).
struct ConvIn {
    const __bf16 *x;
    int C;
    const __bf16 *skip = nullptr;
    int Cs = 0;
};

// the source of the channels from c on: its array at channel c, its channels and
// the shift of the mesh coordinates
struct ConvSrc {
    const __bf16 *x;
    int C, sh;
};

__device__ __forceinline__ ConvSrc conv_src(const ConvIn &I, int c)
{
    if (!I.skip) return ConvSrc{I.x + c, I.C, 0};
    return c < I.C ? ConvSrc{I.x + c, I.C, 1} : ConvSrc{I.skip + (c - I.C), I.Cs, 0};
}

// The same convolution for S >= 16 and input channels in chunks of CK = 16 or 32
// (every layer of the network above the 8^3 mesh, and their backward-data passes).
//
// A workgroup computes 16 NT output channels (those of blockIdx.y) and walks over
// tiles of 16 x 8 x TZ voxels; each of its waves keeps the weight fragments of
// 16 channels and one chunk in registers (14 k-steps of two taps each, or 27 of
// one; with one chunk they are loaded once) and takes MT = 2 TZ NT rows of 16
// voxels.  The next tile's (chunk's) halo block is loaded into registers while the
// current one is multiplied.  Operands are swapped against k_conv3d, so that a
// lane ends with four consecutive channels of one voxel and stores them at once;
// the products and their order are the same, and so are the results.  LDS holds
// the CK / 8 parts of 8 channels of the block apart, 16 bytes per voxel, each part
// starting a multiple of 256 bytes on: the lanes of a fragment read, and those of
// a staging write, take 256 contiguous bytes.  The address of every fragment is a
// per-lane base (for CK = 16 one of three: the distance of a k-step's two taps
// takes three values) plus a constant.
// Fragments are shared between the rows (CK = 32: an input row's three serve three
// output rows, 30 reads of LDS for 72 products) or planes (CK = 16) of a wave.
// Bound: the halo traffic and the staging between products; 16 -> 16 channels move
// 134 MB of HBM in 40 us (3.3 TB/s) with the matrix cores a third busy.
// us, before (weights from L1 in every k-step, two-way bank conflicts, no loads in
// flight during the products, two-byte stores) and now, 2.1 M voxels: 16 -> 16
// channels 110, 40; 48 -> 16 340, 111; 16 -> 48 176, 127; 262144 voxels: 16 -> 32
// 25, 14; 32 -> 32 46, 20; 96 -> 32 120, 50; 32 -> 96 114, 45; 32 -> 16 41, 15;
// 32768 voxels: 32 -> 64 22, 7.7; 64 -> 64 39, 17; 64 -> 32 34, 14.
template <int CK, int NT, int TZ, bool MASK, bool SKIP>
__global__ __launch_bounds__(256, 2) void k_conv_reg(ConvIn in, int lgS, const __bf16 *__restrict__ W,
                                                     const float *__restrict__ bias, int Cout, int relu,
                                                     const __bf16 *__restrict__ M, unsigned ntiles,
                                                     __bf16 *__restrict__ Y, float *__restrict__ Y32)
{
    constexpr int MT = 2 * TZ * NT, HX = 18, HY = 10, HV = HX * HY * (TZ + 2), Q = CK / 8, HP = (HV + 15) / 16 * 16;
    constexpr int NK = CK == 16 ? 14 : 27;
    constexpr int NP = (HP * Q + 255) / 256;  // 16-byte pieces of a halo block per thread
    const int Cin = SKIP ? in.C + in.Cs : in.C;
    static_assert(MT == 4 || MT % 8 == 0, "a wave's rows are half a z-plane of the tile or whole ones");
    __shared__ __attribute__((aligned(16))) __bf16 sX[Q * HP * 8];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, r16 = lane & 15;
    const int S = 1 << lgS, sm = S - 1;
    const unsigned ntx = (unsigned)S / 16, nty = (unsigned)S / 8, ntz = (unsigned)S / TZ;
    // this wave's rows: with PAIR rows 2 w and 2 w + 1 of every plane, else whole planes or half of one
    constexpr bool PAIR = CK == 16 && NT == 1 && TZ == 4 && !MASK;
    const int row0 = (w / NT) * MT, wz = PAIR ? 0 : row0 >> 3, wy = PAIR ? 2 * w : row0 & 7;
    auto rowz = [](int mt) { return PAIR ? mt >> 1 : mt >> 3; };
    auto rowy = [](int mt) { return PAIR ? mt & 1 : mt & 7; };
    const int o0 = 16 * ((int)blockIdx.y * NT + w % NT);            // its output channels
    const __bf16 *p0 = sX + ((g & (Q - 1)) * HP + (wz * HY + wy) * HX + r16) * 8;
    // CK = 16, k-step k: voxel offset of tap 2 k, for lanes of g >= 2 that of tap 2 k + 1
    const __bf16 *pb[3] = {p0 + (g >= 2 ? 8 : 0), p0 + (g >= 2 ? 8 * (HX - 2) : 0),
                           p0 + (g >= 2 ? 8 * (HX * HY - 2 * HX - 2) : 0)};
    const bool pad = g >= 2;  // the second tap of its last k-step does not exist: zeros
    float bo[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) bo[j] = bias ? bias[o0 + 4 * g + j] : 0.f;
    auto origin = [&](unsigned tile, int &x0, int &y0, int &z0, size_t &vol) {
        x0 = (int)(tile % ntx) * 16;
        tile /= ntx;
        y0 = (int)(tile % nty) * 8;
        tile /= nty;
        z0 = (int)(tile % ntz) * TZ;
        vol = (size_t)(tile / ntz) << (3 * lgS);
    };
    // staging: this thread's pieces are part pq of voxels pv + 256 / Q i of the halo
    // block, whose coordinates mod S are kept packed as z, y, x fields of lgS bits
    const int pq = (tid >> 4) & (Q - 1), pv = ((tid >> 4) / Q) * 16 + (tid & 15);
    __bf16 *pst = sX + (pq * HP + pv) * 8;
    const unsigned top = (1u | 1u << lgS | 1u << (2 * lgS)) << (lgS - 1);  // highest bit of each field
    unsigned pc[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        const int v = min(pv + 256 / Q * i, HV - 1);
        const int vx = v % HX, vy = (v / HX) % HY, vz = v / (HX * HY);
        pc[i] = (((((unsigned)(vz & sm)) << lgS) | (unsigned)(vy & sm)) << lgS) | (unsigned)(vx & sm);
    }
    bf16x8 st[NP];
    auto fetch = [&](unsigned tile, int cc0) {
        int x0, y0, z0;
        size_t vol;
        origin(tile, x0, y0, z0, vol);
        const ConvSrc from = SKIP ? conv_src(in, cc0) : ConvSrc{in.x + cc0, in.C, 0};
        const __bf16 *x = from.x + (vol >> (3 * from.sh)) * from.C;
        const unsigned og = (((((unsigned)((z0 - 1) & sm)) << lgS) | (unsigned)((y0 - 1) & sm)) << lgS) |
                            (unsigned)((x0 - 1) & sm);
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            // the fields' sums mod S: carries stop below the highest bits, which add without
            unsigned r = ((pc[i] & ~top) + (og & ~top)) ^ ((pc[i] ^ og) & top);
            if (SKIP && from.sh) {
                const int lc = lgS - 1;
                r = ((((r >> (2 * lgS + 1)) << lc) | ((r >> (lgS + 1)) & (unsigned)(sm >> 1))) << lc) |
                    ((r >> 1) & (unsigned)(sm >> 1));
            }
            st[i] = *(const bf16x8 *)(x + (size_t)r * from.C + 8 * pq);
        }
    };
    bf16x8 b[NK];
    const unsigned woff = (unsigned)((o0 + r16) * Cin + 8 * (g & (Q - 1))), woff2 = woff + (g >= 2 ? (unsigned)(Cout * Cin) : 0);
    auto weights = [&](int cc0) {
        const int tap = Cout * Cin;
#pragma unroll
        for (int k = 0; k < NK; ++k) {
            const bool last = CK == 16 && k == NK - 1;
            const __bf16 *wk = W + (CK == 16 ? 2 * k : k) * tap + cc0;  // uniform
            b[k] = *(const bf16x8 *)(wk + (CK == 32 || last ? woff : woff2));
            if (last) b[k] = pad ? bf16x8{} : b[k];
        }
    };
    const unsigned lo = (unsigned)(r16 * Cout + 4 * g);  // this lane's place in an output row
    if (Cin == CK) weights(0);
    if (blockIdx.x < ntiles) fetch(blockIdx.x, 0);
    for (unsigned tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        f32x4 acc[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
        int x0, y0, z0;
        size_t vol;
        origin(tile, x0, y0, z0, vol);
        auto out_row = [&](int mt) {  // uniform
            return (vol + ((((size_t)(z0 + wz + rowz(mt)) << lgS) + (size_t)(y0 + wy + rowy(mt))) << lgS) + (size_t)x0) *
                       Cout + o0;
        };
        bf16x4 m[MT] = {};
        if (MASK && CK == 16)  // in flight during the products (for CK = 32 the registers do not allow it)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) m[mt] = *(const bf16x4 *)(M + out_row(mt) + lo);
        for (int cc0 = 0; cc0 < Cin; cc0 += CK) {
            if (Cin > CK) weights(cc0);
            __syncthreads();  // the previous block's readers are done
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                if (pv + 256 / Q * i < HP) *(bf16x8 *)(pst + 256 / Q * i * 8) = st[i];
            }
            __syncthreads();
            const bool more = cc0 + CK < Cin;
            const unsigned next = more ? tile : tile + gridDim.x;
            if (next < ntiles) fetch(next, more ? cc0 + CK : 0);
            if constexpr (CK == 32) {
                // Input row by input row: its three fragments (dx) serve the rows y
                // - dy of the wave; every row's sum still runs over dz, dy, dx in turn
                constexpr int RY = MT == 8 ? 8 : MT, IR = RY + 2;
                bf16x8 f[2][3];
                auto rowload = [&](int r, bf16x8 *d) {
#pragma unroll
                    for (int dx = 0; dx < 3; ++dx)
                        d[dx] = *(const bf16x8 *)(p0 + (((r / IR) * HY + r % IR) * HX + dx) * 8);
                };
                rowload(0, f[0]);
#pragma unroll
                for (int r = 0; r < 3 * IR; ++r) {
                    __builtin_amdgcn_sched_barrier(0);  // reads of later rows would spill (and 10 % slower without)
                    if (r + 1 < 3 * IR) rowload(r + 1, f[(r + 1) & 1]);
#pragma unroll
                    for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                        for (int dy = 0; dy < 3; ++dy) {
                            const int y = r % IR - dy;
                            if (y >= 0 && y < RY)
                                acc[y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[(r / IR) * 9 + dy * 3 + dx], f[r & 1][dx],
                                                                                 acc[y], 0, 0, 0);
                        }
                }
            } else if constexpr (PAIR) {
                // Input plane by input plane: fragments of taps (dx 0, 1), (1, 2) and (2, 0 of
                // the next row) serve up to three planes of the wave; every row's sum still
                // runs over the k-steps in turn
                auto frag = [&](const __bf16 *base, int zi, int y, int dx) {
                    return *(const bf16x8 *)(base + ((zi * HY + y) * HX + dx) * 8);
                };
                auto mul = [&](int k, const bf16x8 &a, int z, int y) {
                    acc[2 * z + y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[k], a, acc[2 * z + y], 0, 0, 0);
                };
#pragma unroll
                for (int zi = 0; zi < TZ + 2; ++zi) {
                    bf16x8 A[4], B[3], C[4], D[2] = {}, E[2] = {};
                    const bool top = zi < TZ, mid = zi > 0 && zi <= TZ, bot = zi > 1;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        A[r] = frag(pb[0], zi, r, 0);
                        C[r] = frag(pb[0], zi, r, 1);
                        if (r < 3) B[r] = frag(pb[1], zi, r, 2);
                    }
#pragma unroll
                    for (int y = 0; y < 2; ++y) {
                        if (top) D[y] = frag(pb[2], zi, y + 2, 2);
                        if (bot) E[y] = pad ? bf16x8{} : frag(p0, zi, y + 2, 2);
                    }
#pragma unroll
                    for (int i = 0; i < 5; ++i)
#pragma unroll
                        for (int y = 0; y < 2; ++y) {
                            const bf16x8 t = i == 0 ? A[y] : i == 1 ? B[y] : i == 2 ? C[y + 1] : i == 3 ? A[y + 2] : D[y];
                            const bf16x8 m = i == 0 ? C[y] : i == 1 ? A[y + 1] : i == 2 ? B[y + 1] : C[y + 2];
                            const bf16x8 o = i == 0 ? A[y] : i == 1 ? B[y] : i == 2 ? C[y + 1] : i == 3 ? A[y + 2] : E[y];
                            if (top) mul(i, t, zi, y);
                            if (mid && i < 4) mul(5 + i, m, zi - 1, y);
                            if (bot) mul(9 + i, o, zi - 2, y);
                        }
                }
            } else {
#pragma unroll
                for (int k = 0; k < NK; ++k) {
                    const int t = 2 * k;  // compile-time: the loop is unrolled
                    const __bf16 *q = (t == 26 ? p0 : pb[t % 3 != 2 ? 0 : t % 9 != 8 ? 1 : 2]) +
                                      (((t / 9) * HY + (t / 3) % 3) * HX + t % 3) * 8;
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        bf16x8 a = *(const bf16x8 *)(q + mt * HX * 8);
                        if (k == NK - 1) a = pad ? bf16x8{} : a;
                        acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[k], a, acc[mt], 0, 0, 0);
                    }
                }
            }
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const size_t row = out_row(mt);
            float o[4];
            if (MASK && CK == 32) m[mt] = *(const bf16x4 *)(M + row + lo);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                o[j] = acc[mt][j] + bo[j];
                if (relu) o[j] = fmaxf(o[j], 0.f);
                if (MASK && !(bf2f(m[mt][j]) > 0.f)) o[j] = 0.f;
            }
            if (Y) *(bf16x4 *)(Y + row + lo) = bf16x4{f2bf(o[0]), f2bf(o[1]), f2bf(o[2]), f2bf(o[3])};
            if (Y32) *(f32x4 *)(Y32 + row + lo) = f32x4{o[0], o[1], o[2], o[3]};
        }
    }
}

// Launch k_conv_reg or k_conv3d over nvox = B S^3 voxels (S >= 8, Cout a multiple of 16 up to 96).
// With a mask M (Cout channels, for a gradient through a ReLU) Y is zero where M > 0 does not hold.
// A skip connection is for the shapes of the decoder's layers: meshes of 16^3 and up, 32 + 16 to
// 16 channels or both multiples of 32 to a multiple of 32, no mask; others are refused.
int launch_conv3d(const ConvIn &in, size_t nvox, int lgS, const __bf16 *W, const float *bias, int Cout, int relu,
                  const __bf16 *M, __bf16 *Y, float *Y32, hipStream_t s)
{
    const int Cin = in.C + in.Cs;
    // k_conv_reg stores four channels at once; outputs off those boundaries take k_conv3d
    const bool aligned = ((uintptr_t)Y & 7) == 0 && ((uintptr_t)Y32 & 15) == 0;
    const bool reg = Cin % 16 == 0 && lgS >= 4 && aligned;
    const int CK = Cin % 32 == 0 ? 32 : 16;
    // two blocks of 16 channels per workgroup where the number is even: its
    // weights still fit in the registers and the input is read half as often
    const int NT = Cout % 32 == 0 ? 2 : 1;
    if (in.skip && (!reg || M || in.C % CK || NT != CK / 16))
        return set_error(MGFR_ERR_ARG, "no convolution of two sources with %d + %d to %d channels here", in.C, in.Cs, Cout);
    if (reg) {
        const unsigned groups = (unsigned)(Cout / (16 * NT));
        // persistent, two workgroups per CU (their registers; 768 groups on 512
        // places: 59 us instead of 49 for 16 -> 16 channels)
        auto go = [&](auto *k, unsigned tz) {
            const unsigned nt = (unsigned)(nvox / (128 * tz));
            k<<<dim3(std::min(nt, std::max(512u / groups, 1u)), groups), 256, 0, s>>>(in, lgS, W, bias, Cout, relu,
                                                                                      M, nt, Y, Y32);
        };
        auto pick = [&](auto *masked, auto *plain, unsigned tz) { M ? go(masked, tz) : go(plain, tz); };
        // The deepest tile that the registers allow loads the fewest voxels of halo
        // (4 planes: 2.1 per voxel, 2: 2.8, 1: 4.2); a shallower one where the
        // tiles would leave CUs without a workgroup
        const size_t b4 = nvox / 512 * groups, b2 = nvox / 256 * groups;
        if (in.skip && CK == 32)
            b2 >= 256 ? go(k_conv_reg<32, 2, 2, false, true>, 2) : go(k_conv_reg<32, 2, 1, false, true>, 1);
        else if (in.skip)
            b4 >= 256 ? go(k_conv_reg<16, 1, 4, false, true>, 4) : go(k_conv_reg<16, 1, 2, false, true>, 2);
        else if (CK == 32) {
            if (NT == 1)
                pick(k_conv_reg<32, 1, 2, true, false>, k_conv_reg<32, 1, 2, false, false>, 2);
            else if (b2 >= 256)
                pick(k_conv_reg<32, 2, 2, true, false>, k_conv_reg<32, 2, 2, false, false>, 2);
            else
                pick(k_conv_reg<32, 2, 1, true, false>, k_conv_reg<32, 2, 1, false, false>, 1);
        } else if (NT == 1) {
            if (b4 >= 256)
                pick(k_conv_reg<16, 1, 4, true, false>, k_conv_reg<16, 1, 4, false, false>, 4);
            else
                pick(k_conv_reg<16, 1, 2, true, false>, k_conv_reg<16, 1, 2, false, false>, 2);
        } else if (b2 >= 256)
            pick(k_conv_reg<16, 2, 2, true, false>, k_conv_reg<16, 2, 2, false, false>, 2);
        else
            pick(k_conv_reg<16, 2, 1, true, false>, k_conv_reg<16, 2, 1, false, false>, 1);
        MGFR_HIP(hipGetLastError());
        return MGFR_OK;
    }
    const unsigned blocks = (unsigned)(nvox / (16 * kConvMT * kConvWaves));
    // LDS: the halo tile ((TX+2) x 10 x (TZ+2) voxels) times the channel chunk (bf16)
    const int TX = lgS < 4 ? (1 << lgS) : 16, TZ = (16 * kConvMT * kConvWaves) / (TX * 8);
    const int CC = (Cin % 32 == 0) ? 32 : ((Cin % 16 == 0) ? 16 : 8);
    const size_t lds = (size_t)(TX + 2) * 10 * (TZ + 2) * conv_stride(CC) * sizeof(__bf16);
    int nt = Cout >> 4, groups = 1;
    // fewer than two workgroups per CU: split the output channels
    while (blocks * groups < 512 && nt % 2 == 0) {
        nt /= 2;
        groups *= 2;
    }
    const dim3 grid(blocks, groups);
    switch (nt) {
    case 1: k_conv3d<1><<<grid, 64 * kConvWaves, lds, s>>>(in.x, lgS, Cin, W, bias, Cout, relu, M, Y, Y32); break;
    case 2: k_conv3d<2><<<grid, 64 * kConvWaves, lds, s>>>(in.x, lgS, Cin, W, bias, Cout, relu, M, Y, Y32); break;
    case 3: k_conv3d<3><<<grid, 64 * kConvWaves, lds, s>>>(in.x, lgS, Cin, W, bias, Cout, relu, M, Y, Y32); break;
    case 4: k_conv3d<4><<<grid, 64 * kConvWaves, lds, s>>>(in.x, lgS, Cin, W, bias, Cout, relu, M, Y, Y32); break;
    case 5: k_conv3d<5><<<grid, 64 * kConvWaves, lds, s>>>(in.x, lgS, Cin, W, bias, Cout, relu, M, Y, Y32); break;
    default: k_conv3d<6><<<grid, 64 * kConvWaves, lds, s>>>(in.x, lgS, Cin, W, bias, Cout, relu, M, Y, Y32); break;
    }
    MGFR_HIP(hipGetLastError());
    return MGFR_OK;
}

// dW[t][o][c] += sum_v dZ[v][o] X[v + off(t)][c] and db[o] += sum_v dZ[v][o];
// Cin, Cout % 16 == 0, S >= 8.
//
// A GEMM per tap whose reduction runs over voxels, with both operands stored
// channels-last, i.e. the wrong way round for the MFMA fragments (8
// consecutive k = voxels per lane).  A workgroup owns one 16 x 16 block of
// (output, input) channels for all 27 taps and walks over tiles of 512
// voxels (TX x 8 x TZ): the tile of dZ and the tile plus halo of X are staged
// once, as they lie in memory, and every tap's fragments are read from there
// by the LDS transpose load (ds_read_b64_tr_b16: 16 lanes read 4 voxels x 16
// channels and get 4 voxels of one channel each).  The order of the voxels
// within a k-step is free, as long as both operands use the same: the 16
// lanes of a group and the two halves of a fragment are laid out so that one
// load of a wave reads 16 consecutive voxels of a row (512 contiguous bytes,
// no bank conflict).  Wave w accumulates the columns of taps (dz, dx) number w,
// w + 4, w + 8 (the fourth wave the bias gradient, a product with ones, beside its
// two); the three taps dy of a column share their rows, so that a k-step reads two
// new half fragments per column instead of six.  The sums stay in registers over
// all tiles and are added to dW once per workgroup; the next tile is loaded into
// registers during the products.  The caller's x and dZ may start at any element.
// Bound: the traffic (16 -> 16 channels on 2.1 M voxels: 134 MB and the halos) and
// the barriers around the staging.  That layer: 2163 us with a scalar transpose
// into LDS per tap; 87 with transpose loads; 67 with the next tile in flight; 61
// with shared rows (475 TFLOP/s).  The ten layers of one gradient of eight 64^3
// volumes: 14.4 -> 0.52 ms, and a separate bias pass's 3.9 ms are gone.
#ifndef MGFR_WG_SPLIT
#define MGFR_WG_SPLIT 512
#endif
constexpr int kWgTile = 512;
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

__device__ __forceinline__ s16x4 tr_half(const __bf16 *p)
{
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)p);
}

__device__ __forceinline__ bf16x8 join(s16x4 lo, s16x4 hi)
{
    const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
}

// grid (Cout / 16 * Cin / 16, splits of the tiles)
template <int LGX>
__global__ __launch_bounds__(256) void k_conv3d_wgrad(ConvIn in, const __bf16 *__restrict__ dZ, int lgS, int Cout,
                                                       unsigned ntiles, float *__restrict__ dW, float *__restrict__ db)
{
    const int Cin = in.C + in.Cs;
    constexpr int TX = 1 << LGX, TZ = kWgTile / (8 * TX);
    constexpr int HX = TX + 2, HY = 10, HV = HX * HY * (TZ + 2);
    __shared__ __attribute__((aligned(16))) __bf16 sX[HV * 16];
    __shared__ __attribute__((aligned(16))) __bf16 sZ[kWgTile * 16];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, r16 = lane & 15;
    const int S = 1 << lgS, sm = S - 1;
    const int CT = Cin >> 4;
    const int o0 = 16 * ((int)blockIdx.x / CT), c0 = 16 * ((int)blockIdx.x % CT);
    const bool bias = db != nullptr && c0 == 0 && w == 3;
    const ConvSrc from = conv_src(in, c0);
    const unsigned ntx = (unsigned)S / TX, nty = (unsigned)S / 8, ntz = (unsigned)S / TZ;
    // this lane's part of a row of voxels: voxel 4 g + r16 / 4 of 16, channels 4 (r16 & 3) ..
    const int v0 = 4 * g + (r16 >> 2), c4 = 4 * (r16 & 3);
    const __bf16 *pz = sZ + v0 * 16 + c4;
    const __bf16 *px = sX + (((HY + 1 + (v0 >> LGX)) * HX) + 1 + (v0 & (TX - 1))) * 16 + c4;
    // the wave's columns of taps (dz, dx): 9 over four waves; [..][dy]
    const bool third = w == 0;
    f32x4 acc[3][3] = {};
    const __bf16 *pt[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const int c = q < 2 || third ? w + 4 * q : 0;
        pt[q] = px + ((c / 3 - 1) * HY * HX + (c % 3 - 1)) * 16;
    }
    const __bf16 one = (__bf16)1.0f;
    const bf16x8 ones = {one, one, one, one, one, one, one, one};
    // staging: 16-byte pieces, half h of voxel sv + 128 i of the tile (dZ) and of the
    // halo block (X), the latter's coordinates mod S packed as z, y, x fields
    constexpr int PZ = kWgTile * 2 / 256, PX = (HV * 2 + 255) / 256;
    const int sv = tid >> 1, h8 = 8 * (tid & 1);
    const unsigned zoff = (((((unsigned)sv >> (LGX + 3)) << lgS) + ((sv >> LGX) & 7)) << lgS) + (sv & (TX - 1));
    const unsigned top = (1u | 1u << lgS | 1u << (2 * lgS)) << (lgS - 1);  // highest bit of each field
    unsigned pc[PX];
#pragma unroll
    for (int i = 0; i < PX; ++i) {
        const int v = min(sv + 128 * i, HV - 1), x = v % HX, y = (v / HX) % HY, z = v / (HX * HY);
        pc[i] = ((((unsigned)(z & sm) << lgS) | (unsigned)(y & sm)) << lgS) | (unsigned)(x & sm);
    }
    bf16x8 rz[PZ], rx[PX];
    auto fetch = [&](unsigned b) {
        const int x0 = (int)(b % ntx) * TX;
        b /= ntx;
        const int y0 = (int)(b % nty) * 8;
        b /= nty;
        const int z0 = (int)(b % ntz) * TZ;
        const size_t vol = (size_t)(b / ntz) << (3 * lgS);
        const size_t org = vol + ((((size_t)z0 << lgS) + (size_t)y0) << lgS) + (size_t)x0;
        const __bf16 *z = dZ + org * Cout + o0, *x = from.x + (vol >> (3 * from.sh)) * from.C;
        const unsigned og = ((((unsigned)((z0 - 1) & sm) << lgS) | (unsigned)((y0 - 1) & sm)) << lgS) |
                            (unsigned)((x0 - 1) & sm);
#pragma unroll
        for (int i = 0; i < PZ; ++i)
            rz[i] = *(const bf16x8_any *)(z + ((size_t)(i * 16 / TX) << (2 * lgS)) * Cout + (size_t)zoff * Cout + h8);
#pragma unroll
        for (int i = 0; i < PX; ++i) {
            // the fields' sums mod S: carries stop below the highest bits, which add without
            unsigned r = ((pc[i] & ~top) + (og & ~top)) ^ ((pc[i] ^ og) & top);
            if (from.sh) {
                const int lc = lgS - 1;
                r = ((((r >> (2 * lgS + 1)) << lc) | ((r >> (lgS + 1)) & (unsigned)(sm >> 1))) << lc) |
                    ((r >> 1) & (unsigned)(sm >> 1));
            }
            rx[i] = *(const bf16x8_any *)(x + (size_t)r * from.C + h8);
        }
    };
    if (blockIdx.y < ntiles) fetch(blockIdx.y);
    for (unsigned tile = blockIdx.y; tile < ntiles; tile += gridDim.y) {
        __syncthreads();  // the previous tile's readers are done
#pragma unroll
        for (int i = 0; i < PZ; ++i) *(bf16x8 *)(sZ + (sv + 128 * i) * 16 + h8) = rz[i];
#pragma unroll
        for (int i = 0; i < PX; ++i)
            if (sv + 128 * i < HV) *(bf16x8 *)(sX + (sv + 128 * i) * 16 + h8) = rx[i];
        __syncthreads();
        if (tile + gridDim.y < ntiles) fetch(tile + gridDim.y);
        // k-steps of 32 voxels: two halves of 16, each one row of 16 or two rows of 8
        constexpr int RG = 16 / TX, KP = 4 / RG;  // rows per half, k-steps per plane
        for (int z = 0; z < TZ; ++z) {
            auto half = [&](int q, int row) { return tr_half(pt[q] + (z * HY + row) * HX * 16); };
            s16x4 h[3][4];  // RG = 1: rows 2 ks - 1 .. 2 ks + 2 of each column
            if constexpr (RG == 1) {
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    if (q < 2 || third) {
                        h[q][2] = half(q, -1);
                        h[q][3] = half(q, 0);
                    }
            }
#pragma unroll
            for (int ks = 0; ks < KP; ++ks) {
                const __bf16 *za = pz + (z * KP + ks) * 512;
                const bf16x8 a = join(tr_half(za), tr_half(za + 256));
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    if (q < 2 || third) {
                        if constexpr (RG == 1) {
                            h[q][0] = h[q][2];
                            h[q][1] = h[q][3];
                            h[q][2] = half(q, 2 * ks + 1);
                            h[q][3] = half(q, 2 * ks + 2);
                        }
#pragma unroll
                        for (int dy = 0; dy < 3; ++dy) {
                            const bf16x8 x = RG == 1 ? join(h[q][dy], h[q][dy + 1])
                                                     : join(half(q, 4 * ks + dy - 1), half(q, 4 * ks + dy + 1));
                            acc[q][dy] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, x, acc[q][dy], 0, 0, 0);
                        }
                    }
                if (bias) acc[2][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, ones, acc[2][0], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int dy = 0; dy < 3; ++dy) {
            const int c = w + 4 * q, t = (c / 3) * 9 + dy * 3 + c % 3;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int o = o0 + 4 * g + j;
                if (c < 9) unsafeAtomicAdd(&dW[((size_t)t * Cout + o) * Cin + c0 + r16], acc[q][dy][j]);
                else if (bias && dy == 0 && r16 == 0) unsafeAtomicAdd(&db[o], acc[q][dy][j]);
            }
        }
}

// Launch k_conv3d_wgrad over nvox = B S^3 voxels (a multiple of 512: S >= 8).
// Two workgroups per CU over all channel blocks: each adds a whole channel
// block to dW with atomics, so more of them cost more than they hide (the ten
// layers of a gradient of eight 64^3 volumes with 512, 768 and 1024
// workgroups: 0.60, 0.72 and 0.74 ms).
void launch_wgrad(const ConvIn &in, const __bf16 *dZ, size_t nvox, int lgS, int Cout, float *dW, float *db,
                  hipStream_t s)
{
    const unsigned ntiles = (unsigned)(nvox / kWgTile), pairs = (unsigned)(((in.C + in.Cs) >> 4) * (Cout >> 4));
    const dim3 grid(pairs, std::max(1u, std::min(ntiles, (unsigned)MGFR_WG_SPLIT / pairs)));
    if (lgS == 3)
        k_conv3d_wgrad<3><<<grid, 256, 0, s>>>(in, dZ, lgS, Cout, ntiles, dW, db);
    else
        k_conv3d_wgrad<4><<<grid, 256, 0, s>>>(in, dZ, lgS, Cout, ntiles, dW, db);
}

// Wt[t'][c][o] = W[26 - t'][o][c]: weights of the backward-data convolution
__global__ void k_wt_transpose(const __bf16 *__restrict__ W, int Cin, int Cout, __bf16 *__restrict__ Wt)
{
    const size_t n = (size_t)27 * Cin * Cout;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const int o = (int)(i % Cout);
        const int c = (int)((i / Cout) % Cin);
        const int t = (int)(i / ((size_t)Cout * Cin));
        Wt[i] = W[((size_t)(26 - t) * Cout + o) * Cin + c];
    }
}

// ---------------------------------------------------------------- glue

__global__ void k_features(const double *__restrict__ delta, size_t nvox, int lgS, const float *__restrict__ cond,
                           __bf16 *__restrict__ x0)
{
    for (size_t v = (size_t)blockIdx.x * blockDim.x + threadIdx.x; v < nvox; v += (size_t)gridDim.x * blockDim.x) {
        const size_t b = v >> (3 * lgS);
        bf16x8 lo = bf16x8{}, hi = bf16x8{};
        lo[0] = f2bf((float)(asinh(delta[v]) * 0.25));
        lo[1] = f2bf(cond[2 * b + 0]);
        lo[2] = f2bf(cond[2 * b + 1]);
        *(bf16x8 *)(x0 + v * 16) = lo;
        *(bf16x8 *)(x0 + v * 16 + 8) = hi;
    }
}

// 2^3 mean: out has side S/2 (lgS of the output); 8 channels (16 bytes) per thread
__global__ __launch_bounds__(256) void k_pool(const __bf16 *__restrict__ in, int lgSo, int C, size_t nout,
                                              __bf16 *__restrict__ out)
{
    const int So = 1 << lgSo, sm = So - 1, lgSi = lgSo + 1, C8 = C >> 3;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < nout * C8; i += (size_t)gridDim.x * 256) {
        const int c = 8 * (int)(i % C8);
        const size_t v = i / C8;
        const int x = (int)(v & sm), y = (int)((v >> lgSo) & sm), z = (int)((v >> (2 * lgSo)) & sm);
        const size_t b = v >> (3 * lgSo);
        float s[8] = {};
#pragma unroll
        for (int a = 0; a < 8; ++a) {
            const size_t src = (((b << lgSi) + (2 * z + (a >> 2))) << (2 * lgSi)) + ((size_t)(2 * y + ((a >> 1) & 1)) << lgSi) +
                               (2 * x + (a & 1));
            const bf16x8 d = *(const bf16x8 *)(in + src * C + c);
#pragma unroll
            for (int j = 0; j < 8; ++j) s[j] += bf2f(d[j]);
        }
        bf16x8 o;
#pragma unroll
        for (int j = 0; j < 8; ++j) o[j] = f2bf(0.125f * s[j]);
        *(bf16x8 *)(out + v * C + c) = o;
    }
}

// out[v] = concat(in[parent(v)] (Cu channels), skip[v] (Cs channels)): the
// nearest-neighbour upsampling and the skip connection of one decoder level in
// one pass, 8 channels (16 bytes) per thread; Cu, Cs multiples of 8
__global__ void k_concat_up(const __bf16 *__restrict__ in, int Cu, const __bf16 *__restrict__ skip, int Cs,
                            int lgSo, size_t nout, __bf16 *__restrict__ out)
{
    const int sm = (1 << lgSo) - 1, lgSi = lgSo - 1, q8 = (Cu + Cs) >> 3, qu = Cu >> 3;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < nout * q8; i += (size_t)gridDim.x * blockDim.x) {
        const size_t v = i / q8;
        const int q = (int)(i - v * q8);
        bf16x8 val;
        if (q < qu) {
            const int x = (int)(v & sm), y = (int)((v >> lgSo) & sm), z = (int)((v >> (2 * lgSo)) & sm);
            const size_t b = v >> (3 * lgSo);
            const size_t src = (((b << lgSi) + (z >> 1)) << (2 * lgSi)) + ((size_t)(y >> 1) << lgSi) + (x >> 1);
            val = *(const bf16x8 *)(in + src * Cu + 8 * q);
        } else {
            val = *(const bf16x8 *)(skip + v * Cs + 8 * (q - qu));
        }
        *(bf16x8 *)(out + i * 8) = val;
    }
}

// The gradients below are taken through the ReLU that made y on the way out:
// zero where y > 0 does not hold.  Threads take 8 channels (16 bytes) each.
__device__ __forceinline__ bf16x8 through_relu(const float *d, const __bf16 *y)
{
    const bf16x8 m = *(const bf16x8 *)y;
    bf16x8 o;
#pragma unroll
    for (int j = 0; j < 8; ++j) o[j] = bf2f(m[j]) > 0.f ? f2bf(d[j]) : f2bf(0.f);
    return o;
}

// d_in[parent][c] = (y[parent][c] > 0) sum_children d_out[child][c], c < C of Ctot
__global__ __launch_bounds__(256) void k_upsample_bwd(const __bf16 *__restrict__ dout, int lgSi, int C, size_t nin, int Ctot,
                                                      const __bf16 *__restrict__ y, __bf16 *__restrict__ din)
{
    const int Si = 1 << lgSi, sm = Si - 1, lgSo = lgSi + 1, C8 = C >> 3;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < nin * C8; i += (size_t)gridDim.x * 256) {
        const int c = 8 * (int)(i % C8);
        const size_t v = i / C8;
        const int x = (int)(v & sm), yy = (int)((v >> lgSi) & sm), z = (int)((v >> (2 * lgSi)) & sm);
        const size_t b = v >> (3 * lgSi);
        float s[8] = {};
#pragma unroll
        for (int a = 0; a < 8; ++a) {
            const size_t src = (((b << lgSo) + (2 * z + (a >> 2))) << (2 * lgSo)) +
                               ((size_t)(2 * yy + ((a >> 1) & 1)) << lgSo) + (2 * x + (a & 1));
            const bf16x8 d = *(const bf16x8 *)(dout + src * Ctot + c);
#pragma unroll
            for (int j = 0; j < 8; ++j) s[j] += bf2f(d[j]);
        }
        *(bf16x8 *)(din + v * C + c) = through_relu(s, y + v * C + c);
    }
}

// skip-connection gradient: d_skip[v][c] = (y[v][c] > 0) (d_cat[v][off + c] + d_pool[parent(v)][c] / 8)
__global__ __launch_bounds__(256) void k_skip_grad(const __bf16 *__restrict__ dcat, int Ctot, int off,
                                                   const __bf16 *__restrict__ dpool, int lgS, int C, size_t nvox,
                                                   const __bf16 *__restrict__ y, __bf16 *__restrict__ dskip)
{
    const int S = 1 << lgS, sm = S - 1, lgP = lgS - 1, C8 = C >> 3;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < nvox * C8; i += (size_t)gridDim.x * 256) {
        const int c = 8 * (int)(i % C8);
        const size_t v = i / C8;
        const int x = (int)(v & sm), yy = (int)((v >> lgS) & sm), z = (int)((v >> (2 * lgS)) & sm);
        const size_t b = v >> (3 * lgS);
        const size_t par = (((b << lgP) + (z >> 1)) << (2 * lgP)) + ((size_t)(yy >> 1) << lgP) + (x >> 1);
        const bf16x8 dc = *(const bf16x8 *)(dcat + v * Ctot + off + c), dp = *(const bf16x8 *)(dpool + par * C + c);
        float s[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) s[j] = bf2f(dc[j]) + 0.125f * bf2f(dp[j]);
        *(bf16x8 *)(dskip + v * C + c) = through_relu(s, y + v * C + c);
    }
}

// 1x1 head: y[v] = sum_c h[v][c] wh[c] + bh
__global__ void k_head(const __bf16 *__restrict__ h, size_t nvox, const float *__restrict__ wh, float *__restrict__ y)
{
    for (size_t v = (size_t)blockIdx.x * blockDim.x + threadIdx.x; v < nvox; v += (size_t)gridDim.x * blockDim.x) {
        float s = wh[16];
#pragma unroll
        for (int c = 0; c < 16; ++c) s += bf2f(h[v * 16 + c]) * wh[c];
        y[v] = s;
    }
}

// Loss and the head's backward pass in one: with d = 2 (y - u / kUScale) / n,
// loss[0] += sum (y - u / kUScale)^2 / n, dh[v][c] = (h[v][c] > 0) d wh[c],
// dwh[c] += sum_v d h[v][c], dwh[16] += sum_v d.  The sums are formed per
// workgroup first: atomics on these 18 addresses cost 12 ns each one after
// the other (one per wave and sum: 1.78 ms on 2.1 M voxels; 256 workgroups,
// two instructions each: 36 us, the traffic of h, dh, y and u).
constexpr int kHeadBlocks = 256;
__global__ __launch_bounds__(256) void k_loss_head_bwd(const __bf16 *__restrict__ h, const float *__restrict__ y,
                                                        const double *__restrict__ u, size_t n,
                                                        const float *__restrict__ wh, __bf16 *__restrict__ dh,
                                                        float *__restrict__ dwh, float *__restrict__ loss)
{
    __shared__ float sh[4][18];
    float s[18], w[16];
#pragma unroll
    for (int c = 0; c < 18; ++c) s[c] = 0.f;
#pragma unroll
    for (int c = 0; c < 16; ++c) w[c] = wh[c];
    for (size_t v = (size_t)blockIdx.x * 256 + threadIdx.x; v < n; v += (size_t)gridDim.x * 256) {
        const float e = y[v] - (float)u[v] / kUScale, d = 2.f * e / (float)n;
        s[17] += e * e;
        s[16] += d;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const bf16x8 a = *(const bf16x8 *)(h + v * 16 + 8 * q);
            bf16x8 b;
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                s[8 * q + c] += d * bf2f(a[c]);
                b[c] = bf2f(a[c]) > 0.f ? f2bf(d * w[8 * q + c]) : f2bf(0.f);
            }
            *(bf16x8 *)(dh + v * 16 + 8 * q) = b;
        }
    }
#pragma unroll
    for (int c = 0; c < 18; ++c) {
        float x = s[c];
        for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
        if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6][c] = x;
    }
    __syncthreads();
    if (threadIdx.x < 18) {
        const float x = (sh[0][threadIdx.x] + sh[1][threadIdx.x]) + (sh[2][threadIdx.x] + sh[3][threadIdx.x]);
        if (threadIdx.x < 17) unsafeAtomicAdd(&dwh[threadIdx.x], x);
        else unsafeAtomicAdd(loss, x / (float)n);
    }
}

__global__ void k_to_u(const float *__restrict__ y, size_t n, double *__restrict__ u)
{
    for (size_t v = (size_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (size_t)gridDim.x * blockDim.x)
        u[v] = (double)(y[v] * kUScale);
}

// Adam on float32 master weights (bias-corrected; t = step count >= 1)
__global__ void k_adam(float *__restrict__ p, const float *__restrict__ gr, float *__restrict__ m, float *__restrict__ v,
                       size_t n, float lr, float b1, float b2, float eps, float c1, float c2)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const float gi = gr[i];
        const float mi = b1 * m[i] + (1.f - b1) * gi;
        const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    }
}

__global__ void k_to_bf16(const float *__restrict__ p, size_t n, __bf16 *__restrict__ o)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        o[i] = f2bf(p[i]);
}

__global__ void k_restrict4(const double *__restrict__ fine, int lgc, double *__restrict__ coarse)
{
    const int Nc = 1 << lgc, lgf = lgc + 2;
    const size_t n = (size_t)Nc * Nc * Nc;
    for (size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += (size_t)gridDim.x * blockDim.x) {
        const int K = (int)(t & (Nc - 1)), J = (int)((t >> lgc) & (Nc - 1)), I = (int)(t >> (2 * lgc));
        double s = 0.0;
        for (int a = 0; a < 4; ++a)
            for (int b = 0; b < 4; ++b)
                for (int c = 0; c < 4; ++c) s += fine[cidx(4 * I + a, 4 * J + b, 4 * K + c, lgf)];
        coarse[t] = s / 64.0;
    }
}

// coarse = mean of the 8 daughters (the restriction of Sec. 3.3) of a float64 field
__global__ void k_restrict_mean(const double *__restrict__ fine, int lgc, double *__restrict__ coarse)
{
    const int Nc = 1 << lgc, lgf = lgc + 1;
    const size_t n = (size_t)Nc * Nc * Nc;
    for (size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += (size_t)gridDim.x * blockDim.x) {
        const int K = (int)(t & (Nc - 1)), J = (int)((t >> lgc) & (Nc - 1)), I = (int)(t >> (2 * lgc));
        double s = 0.0;
        for (int a = 0; a < 2; ++a)
            for (int b = 0; b < 2; ++b)
                for (int c = 0; c < 2; ++c) s += fine[cidx(2 * I + a, 2 * J + b, 2 * K + c, lgf)];
        coarse[t] = s * 0.125;
    }
}

// u = P(uc) on the finer mesh: the linear reconstruction (parent value plus
// the central-difference gradient, Sec. 3.3), stored (no clearing pass)
__global__ __launch_bounds__(kBlock) void k_prolong_field_set(double *__restrict__ u, const double *__restrict__ uc,
                                                                int lgc)
{
    const size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x;
    const int K = (int)(t & ((1u << lgc) - 1)), J = (int)((t >> lgc) & ((1u << lgc) - 1)), I = (int)(t >> (2 * lgc));
    const int m = (1 << lgc) - 1, lg = lgc + 1;
    const double v0 = uc[cidx(I, J, K, lgc)];
    const double gx = uc[cidx((I + 1) & m, J, K, lgc)] - uc[cidx((I - 1) & m, J, K, lgc)];
    const double gy = uc[cidx(I, (J + 1) & m, K, lgc)] - uc[cidx(I, (J - 1) & m, K, lgc)];
    const double gz = uc[cidx(I, J, (K + 1) & m, lgc)] - uc[cidx(I, J, (K - 1) & m, lgc)];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                double v = v0;
                v += (a ? 0.125 : -0.125) * gx;
                v += (b ? 0.125 : -0.125) * gy;
                v += (c ? 0.125 : -0.125) * gz;
                u[cidx(2 * I + a, 2 * J + b, 2 * K + c, lg)] = v;
            }
}

inline unsigned gridn(size_t n, unsigned cap = 16384) { return (unsigned)std::min<size_t>((n + 255) / 256, cap); }

}  // namespace

}  // namespace mgfr

using namespace mgfr;

// ================================================================ network

namespace {

struct ConvSpec {
    int cin, cout;
    size_t woff, boff;  // offsets into the parameter vector
};

// layer order: c1a c1b c2a c2b c3a c3b c4a c4b c5a c5b, then the head (16 weights + bias)
const int kLayerCin[10] = {16, 16, 16, 32, 32, 64, 96, 32, 48, 16};
const int kLayerCout[10] = {16, 16, 32, 32, 64, 64, 32, 32, 16, 16};

}  // namespace

struct mgfr_net {
    hipStream_t stream = nullptr;
    size_t maxvox = 0;
    ConvSpec L[10];
    size_t nparam = 0, head_off = 0;
    float *p = nullptr, *g = nullptr, *m = nullptr, *v = nullptr;  // master, grad, Adam moments
    __bf16 *wbf = nullptr;   // bf16 copy of every parameter (conv weights used in [t][o][c] layout)
    __bf16 *wt = nullptr;    // transposed, mirrored conv weights for backward-data (same offsets)
    int step = 0;
    int fwd_B = 0, fwd_lg = 0;  // shape of the last forward pass (0: none yet)
    // activations
    __bf16 *x0, *h1a, *s1, *p1, *h2a, *s2, *p2, *h3a, *h3, *h4a, *h4, *h5a, *h5;
    float *y32, *cond, *loss;
    // gradient scratch
    __bf16 *gA, *gB, *gC, *gD;
    float *hcond = nullptr, *hloss = nullptr;
};

namespace {

int net_alloc(mgfr_net *n)
{
    size_t off = 0;
    for (int i = 0; i < 10; ++i) {
        n->L[i].cin = kLayerCin[i];
        n->L[i].cout = kLayerCout[i];
        n->L[i].woff = off;
        off += (size_t)27 * kLayerCin[i] * kLayerCout[i];
        n->L[i].boff = off;
        off += kLayerCout[i];
    }
    n->head_off = off;
    off += 17;
    n->nparam = off;
    const size_t P = n->nparam;
    MGFR_HIP(hipMalloc(&n->p, P * sizeof(float)));
    MGFR_HIP(hipMalloc(&n->g, P * sizeof(float)));
    MGFR_HIP(hipMalloc(&n->m, P * sizeof(float)));
    MGFR_HIP(hipMalloc(&n->v, P * sizeof(float)));
    MGFR_HIP(hipMalloc(&n->wbf, P * sizeof(__bf16)));
    MGFR_HIP(hipMalloc(&n->wt, P * sizeof(__bf16)));
    const size_t V = n->maxvox, V2 = V / 8, V3 = V / 64;
    auto A = [&](__bf16 **ptr, size_t elems) -> int {
        MGFR_HIP(hipMalloc(ptr, elems * sizeof(__bf16)));
        return MGFR_OK;
    };
    int rc;
    if ((rc = A(&n->x0, V * 16)) || (rc = A(&n->h1a, V * 16)) || (rc = A(&n->s1, V * 16)) ||
        (rc = A(&n->p1, V2 * 16)) || (rc = A(&n->h2a, V2 * 32)) || (rc = A(&n->s2, V2 * 32)) ||
        (rc = A(&n->p2, V3 * 32)) || (rc = A(&n->h3a, V3 * 64)) || (rc = A(&n->h3, V3 * 64)) ||
        (rc = A(&n->h4a, V2 * 32)) || (rc = A(&n->h4, V2 * 32)) || (rc = A(&n->h5a, V * 16)) || (rc = A(&n->h5, V * 16)) ||
        (rc = A(&n->gA, V * 48)) || (rc = A(&n->gB, V2 * 96)) || (rc = A(&n->gC, V * 16)) || (rc = A(&n->gD, V * 16)))
        return rc;
    MGFR_HIP(hipMalloc(&n->y32, V * sizeof(float)));
    MGFR_HIP(hipMalloc(&n->cond, 2 * 4096 * sizeof(float)));
    MGFR_HIP(hipMalloc(&n->loss, sizeof(float)));
    MGFR_HIP(hipHostMalloc(&n->hcond, 2 * 4096 * sizeof(float), hipHostMallocDefault));
    MGFR_HIP(hipHostMalloc(&n->hloss, sizeof(float), hipHostMallocDefault));
    return MGFR_OK;
}

void net_free(mgfr_net *n)
{
    if (!n) return;
    void *ptrs[] = {n->p, n->g, n->m, n->v, n->wbf, n->wt, n->x0, n->h1a, n->s1, n->p1, n->h2a, n->s2, n->p2,
                    n->h3a, n->h3, n->h4a, n->h4, n->h5a, n->h5, n->gA, n->gB, n->gC, n->gD,
                    n->y32, n->cond, n->loss};
    for (void *q : ptrs) (void)hipFree(q);
    if (n->hcond) (void)hipHostFree(n->hcond);
    if (n->hloss) (void)hipHostFree(n->hloss);
    delete n;
}

// refresh the bf16 weights and the backward-data copies from the master weights
int net_refresh(mgfr_net *n)
{
    k_to_bf16<<<gridn(n->nparam), 256, 0, n->stream>>>(n->p, n->nparam, n->wbf);
    for (int i = 0; i < 10; ++i)
        k_wt_transpose<<<gridn((size_t)27 * n->L[i].cin * n->L[i].cout), 256, 0, n->stream>>>(
            n->wbf + n->L[i].woff, n->L[i].cin, n->L[i].cout, n->wt + n->L[i].woff);
    MGFR_HIP(hipGetLastError());
    return MGFR_OK;
}

int conv(mgfr_net *n, const ConvIn &in, size_t nvox, int lgS, int layer, __bf16 *y)
{
    const ConvSpec &L = n->L[layer];
    return launch_conv3d(in, nvox, lgS, n->wbf + L.woff, n->p + L.boff, L.cout, 1, nullptr, y, nullptr, n->stream);
}

// Backward through one convolution: from dz, the gradient before the layer's
// ReLU, and its input, accumulates weight and bias gradients and writes the
// input's gradient dx if non-null, with relu_in through the ReLU that made x.
// (Every gradient passes its ReLU where it is written: a pass of its own over dy,
// y and dz was 44 us of the 110 us that a layer of 16 channels took on 2.1 M voxels.)
int conv_bwd(mgfr_net *n, const __bf16 *dz, const ConvIn &in, size_t nvox, int lgS, int layer, __bf16 *dx, bool relu_in)
{
    const ConvSpec &L = n->L[layer];
    launch_wgrad(in, dz, nvox, lgS, L.cout, n->g + L.woff, n->g + L.boff, n->stream);
    MGFR_HIP(hipGetLastError());
    return dx ? launch_conv3d({dz, L.cout}, nvox, lgS, n->wt + L.woff, nullptr, L.cin, 0, relu_in ? in.x : nullptr, dx,
                              nullptr, n->stream)
              : MGFR_OK;
}

int net_forward(mgfr_net *n, const double *delta, int B, int lgS)
{
    const size_t V = (size_t)B << (3 * lgS), V2 = V / 8, V3 = V / 64;
    int rc;
    n->fwd_B = B;
    n->fwd_lg = lgS;
    MGFR_HIP(hipMemcpyAsync(n->cond, n->hcond, 2 * B * sizeof(float), hipMemcpyHostToDevice, n->stream));
    k_features<<<gridn(V), 256, 0, n->stream>>>(delta, V, lgS, n->cond, n->x0);
    if ((rc = conv(n, {n->x0, 16}, V, lgS, 0, n->h1a)) || (rc = conv(n, {n->h1a, 16}, V, lgS, 1, n->s1))) return rc;
    k_pool<<<gridn(V2 * 2), 256, 0, n->stream>>>(n->s1, lgS - 1, 16, V2, n->p1);
    if ((rc = conv(n, {n->p1, 16}, V2, lgS - 1, 2, n->h2a)) || (rc = conv(n, {n->h2a, 32}, V2, lgS - 1, 3, n->s2)))
        return rc;
    k_pool<<<gridn(V3 * 4), 256, 0, n->stream>>>(n->s2, lgS - 2, 32, V3, n->p2);
    if ((rc = conv(n, {n->p2, 32}, V3, lgS - 2, 4, n->h3a)) || (rc = conv(n, {n->h3a, 64}, V3, lgS - 2, 5, n->h3)))
        return rc;
    if ((rc = conv(n, {n->h3, 64, n->s2, 32}, V2, lgS - 1, 6, n->h4a)) ||
        (rc = conv(n, {n->h4a, 32}, V2, lgS - 1, 7, n->h4)))
        return rc;
    if ((rc = conv(n, {n->h4, 32, n->s1, 16}, V, lgS, 8, n->h5a)) || (rc = conv(n, {n->h5a, 16}, V, lgS, 9, n->h5)))
        return rc;
    k_head<<<gridn(V), 256, 0, n->stream>>>(n->h5, V, n->p + n->head_off, n->y32);
    MGFR_HIP(hipGetLastError());
    return MGFR_OK;
}

// Loss against u_target (into n->loss) and the gradient of every parameter.
int net_backward(mgfr_net *n, const double *u_target, int B, int lgS)
{
    const size_t V = (size_t)B << (3 * lgS), V2 = V / 8, V3 = V / 64;
    int rc;
    MGFR_HIP(hipMemsetAsync(n->g, 0, n->nparam * sizeof(float), n->stream));
    MGFR_HIP(hipMemsetAsync(n->loss, 0, sizeof(float), n->stream));
    // loss and head
    k_loss_head_bwd<<<gridn(V, kHeadBlocks), 256, 0, n->stream>>>(n->h5, n->y32, u_target, V, n->p + n->head_off, n->gC,
                                                                  n->g + n->head_off, n->loss);
    // level 1 decoder: c5b (dz = gC) -> gD; c5a -> d(cat5) in gA [V][48]
    if ((rc = conv_bwd(n, n->gC, {n->h5a, 16}, V, lgS, 9, n->gD, true))) return rc;
    if ((rc = conv_bwd(n, n->gD, {n->h4, 32, n->s1, 16}, V, lgS, 8, n->gA, false))) return rc;
    // h4: sum over children of d(cat5)[:, 0:32] -> gB [V2][32]
    k_upsample_bwd<<<gridn(V2 * 4), 256, 0, n->stream>>>(n->gA, lgS - 1, 32, V2, 48, n->h4, n->gB);
    // level 2 decoder: c4b (dz = gB) -> gD; c4a -> d(cat4) in gB [V2][96]
    if ((rc = conv_bwd(n, n->gB, {n->h4a, 32}, V2, lgS - 1, 7, n->gD, true))) return rc;
    if ((rc = conv_bwd(n, n->gD, {n->h3, 64, n->s2, 32}, V2, lgS - 1, 6, n->gB, false))) return rc;
    // h3: sum over children of d(cat4)[:, 0:64] -> gC [V3][64]
    k_upsample_bwd<<<gridn(V3 * 8), 256, 0, n->stream>>>(n->gB, lgS - 2, 64, V3, 96, n->h3, n->gC);
    // level 3: c3b (dz = gC) -> gD; c3a -> d(p2) in gC
    if ((rc = conv_bwd(n, n->gC, {n->h3a, 64}, V3, lgS - 2, 5, n->gD, true))) return rc;
    if ((rc = conv_bwd(n, n->gD, {n->p2, 32}, V3, lgS - 2, 4, n->gC, false))) return rc;
    // s2: d(cat4)[:, 64:96] + d(p2)/8 -> gD [V2][32]
    k_skip_grad<<<gridn(V2 * 4), 256, 0, n->stream>>>(n->gB, 96, 64, n->gC, lgS - 1, 32, V2, n->s2, n->gD);
    // level 2 encoder: c2b (dz = gD) -> gC; c2a -> d(p1) in gD
    if ((rc = conv_bwd(n, n->gD, {n->h2a, 32}, V2, lgS - 1, 3, n->gC, true))) return rc;
    if ((rc = conv_bwd(n, n->gC, {n->p1, 16}, V2, lgS - 1, 2, n->gD, false))) return rc;
    // s1: d(cat5)[:, 32:48] + d(p1)/8 -> gC [V][16]
    k_skip_grad<<<gridn(V * 2), 256, 0, n->stream>>>(n->gA, 48, 32, n->gD, lgS, 16, V, n->s1, n->gC);
    // level 1 encoder: c1b (dz = gC) -> gD; c1a (no input gradient)
    if ((rc = conv_bwd(n, n->gC, {n->h1a, 16}, V, lgS, 1, n->gD, true))) return rc;
    if ((rc = conv_bwd(n, n->gD, {n->x0, 16}, V, lgS, 0, nullptr, false))) return rc;
    MGFR_HIP(hipGetLastError());
    return MGFR_OK;
}

int check_shape(const mgfr_net *n, int B, int S, int *lgS)
{
    if (B < 1 || S < 32 || S > 1024 || (S & (S - 1)))
        return set_error(MGFR_ERR_ARG, "network inputs need B >= 1 and a power-of-two side 32 <= S <= 1024");
    int lg = 0;
    while ((1 << lg) < S) ++lg;
    if (((size_t)B << (3 * lg)) > n->maxvox) return set_error(MGFR_ERR_ARG, "B * S^3 exceeds the network's capacity");
    if (B > 4096) return set_error(MGFR_ERR_ARG, "B must be <= 4096");
    *lgS = lg;
    return MGFR_OK;
}

void set_cond(mgfr_net *n, const double *cond, int B)
{
    for (int b = 0; b < B; ++b) {
        n->hcond[2 * b + 0] = (float)((cond[2 * b + 0] - 0.75) * 4.0);
        n->hcond[2 * b + 1] = (float)((std::log10(cond[2 * b + 1]) + 5.5) / 1.5);
    }
}

}  // namespace

extern "C" int mgfr_net_create(int seed, int64_t max_voxels, void *stream, mgfr_net **out)
{
    if (!out) return set_error(MGFR_ERR_ARG, "out is NULL");
    *out = nullptr;
    if (max_voxels < 4096 || max_voxels % 4096) return set_error(MGFR_ERR_ARG, "max_voxels must be a positive multiple of 4096");
    mgfr_net *n = new (std::nothrow) mgfr_net();
    if (!n) return set_error(MGFR_ERR_OOM, "host allocation failed");
    n->stream = (hipStream_t)stream;
    n->maxvox = (size_t)max_voxels;
    int rc = net_alloc(n);
    if (rc) {
        net_free(n);
        return rc;
    }
    // He-normal initialisation from a seeded generator, zero biases
    std::vector<float> h(n->nparam, 0.f);
    std::mt19937_64 gen((uint64_t)seed);
    for (int i = 0; i < 10; ++i) {
        std::normal_distribution<float> d(0.f, std::sqrt(2.f / (27.f * n->L[i].cin)));
        for (size_t k = 0; k < (size_t)27 * n->L[i].cin * n->L[i].cout; ++k) h[n->L[i].woff + k] = d(gen);
    }
    std::normal_distribution<float> dh(0.f, std::sqrt(1.f / 16.f));
    for (int c = 0; c < 16; ++c) h[n->head_off + c] = dh(gen);
    hipError_t e = hipMemcpy(n->p, h.data(), n->nparam * sizeof(float), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemset(n->m, 0, n->nparam * sizeof(float));
    if (e == hipSuccess) e = hipMemset(n->v, 0, n->nparam * sizeof(float));
    if (e != hipSuccess) {
        net_free(n);
        return hip_fail(e, "network initialisation", __FILE__, __LINE__);
    }
    if ((rc = net_refresh(n))) {
        net_free(n);
        return rc;
    }
    *out = n;
    return MGFR_OK;
}

extern "C" void mgfr_net_destroy(mgfr_net *n) { net_free(n); }

extern "C" int mgfr_net_set_stream(mgfr_net *n, void *stream)
{
    if (!n) return set_error(MGFR_ERR_ARG, "net is NULL");
    n->stream = (hipStream_t)stream;
    return MGFR_OK;
}

extern "C" int64_t mgfr_net_num_params(const mgfr_net *n) { return n ? (int64_t)n->nparam : -1; }

extern "C" int mgfr_net_get_params(mgfr_net *n, float *host)
{
    if (!n || !host) return set_error(MGFR_ERR_ARG, "net and host must be non-NULL");
    MGFR_HIP(hipMemcpyAsync(host, n->p, n->nparam * sizeof(float), hipMemcpyDeviceToHost, n->stream));
    MGFR_HIP(hipStreamSynchronize(n->stream));
    return MGFR_OK;
}

extern "C" int mgfr_net_set_params(mgfr_net *n, const float *host)
{
    if (!n || !host) return set_error(MGFR_ERR_ARG, "net and host must be non-NULL");
    MGFR_HIP(hipMemcpyAsync(n->p, host, n->nparam * sizeof(float), hipMemcpyHostToDevice, n->stream));
    MGFR_HIP(hipMemsetAsync(n->m, 0, n->nparam * sizeof(float), n->stream));
    MGFR_HIP(hipMemsetAsync(n->v, 0, n->nparam * sizeof(float), n->stream));
    n->step = 0;
    int rc = net_refresh(n);
    if (rc) return rc;
    MGFR_HIP(hipStreamSynchronize(n->stream));
    return MGFR_OK;
}

// Checkpoint file: 8-byte tag "MGFRNET1", int64 parameter count, int32 Adam
// step, int32 layer count (10) and each layer's (Cin, Cout) as int32, then the
// float32 master parameters, Adam first and second moments (native byte order).
namespace {
constexpr char kNetTag[8] = {'M', 'G', 'F', 'R', 'N', 'E', 'T', '1'};
}

extern "C" int mgfr_net_save(mgfr_net *n, const char *path)
{
    if (!n || !path) return set_error(MGFR_ERR_ARG, "net and path must be non-NULL");
    const size_t P = n->nparam;
    std::vector<float> buf(3 * P);
    MGFR_HIP(hipMemcpyAsync(buf.data(), n->p, P * sizeof(float), hipMemcpyDeviceToHost, n->stream));
    MGFR_HIP(hipMemcpyAsync(buf.data() + P, n->m, P * sizeof(float), hipMemcpyDeviceToHost, n->stream));
    MGFR_HIP(hipMemcpyAsync(buf.data() + 2 * P, n->v, P * sizeof(float), hipMemcpyDeviceToHost, n->stream));
    MGFR_HIP(hipStreamSynchronize(n->stream));
    FILE *f = fopen(path, "wb");
    if (!f) return set_error(MGFR_ERR_ARG, "cannot open %s for writing", path);
    const int64_t np = (int64_t)P;
    int32_t hdr[2 + 20];
    hdr[0] = n->step;
    hdr[1] = 10;
    for (int i = 0; i < 10; ++i) {
        hdr[2 + 2 * i] = n->L[i].cin;
        hdr[3 + 2 * i] = n->L[i].cout;
    }
    const bool ok = fwrite(kNetTag, 1, 8, f) == 8 && fwrite(&np, sizeof np, 1, f) == 1 &&
                    fwrite(hdr, sizeof hdr, 1, f) == 1 && fwrite(buf.data(), sizeof(float), buf.size(), f) == buf.size();
    if (fclose(f) != 0 || !ok) return set_error(MGFR_ERR_ARG, "writing %s failed", path);
    return MGFR_OK;
}

extern "C" int mgfr_net_load(mgfr_net *n, const char *path)
{
    if (!n || !path) return set_error(MGFR_ERR_ARG, "net and path must be non-NULL");
    FILE *f = fopen(path, "rb");
    if (!f) return set_error(MGFR_ERR_ARG, "cannot open %s", path);
    char tag[8];
    int64_t np = 0;
    int32_t hdr[2 + 20];
    const size_t P = n->nparam;
    std::vector<float> buf(3 * P);
    bool ok = fread(tag, 1, 8, f) == 8 && memcmp(tag, kNetTag, 8) == 0 && fread(&np, sizeof np, 1, f) == 1 &&
              np == (int64_t)P && fread(hdr, sizeof hdr, 1, f) == 1 && hdr[1] == 10;
    for (int i = 0; ok && i < 10; ++i) ok = hdr[2 + 2 * i] == n->L[i].cin && hdr[3 + 2 * i] == n->L[i].cout;
    ok = ok && fread(buf.data(), sizeof(float), buf.size(), f) == buf.size();
    fclose(f);
    if (!ok) return set_error(MGFR_ERR_ARG, "%s is not a checkpoint of this network", path);
    MGFR_HIP(hipMemcpyAsync(n->p, buf.data(), P * sizeof(float), hipMemcpyHostToDevice, n->stream));
    MGFR_HIP(hipMemcpyAsync(n->m, buf.data() + P, P * sizeof(float), hipMemcpyHostToDevice, n->stream));
    MGFR_HIP(hipMemcpyAsync(n->v, buf.data() + 2 * P, P * sizeof(float), hipMemcpyHostToDevice, n->stream));
    n->step = hdr[0];
    int rc = net_refresh(n);
    if (rc) return rc;
    MGFR_HIP(hipStreamSynchronize(n->stream));
    return MGFR_OK;
}

extern "C" int mgfr_net_predict(mgfr_net *n, const double *delta, int B, int S, const double *cond, double *u)
{
    if (!n || !delta || !cond || !u) return set_error(MGFR_ERR_ARG, "net, delta, cond and u must be non-NULL");
    int lgS, rc;
    if ((rc = check_shape(n, B, S, &lgS))) return rc;
    set_cond(n, cond, B);
    if ((rc = net_forward(n, delta, B, lgS))) return rc;
    const size_t V = (size_t)B << (3 * lgS);
    k_to_u<<<gridn(V), 256, 0, n->stream>>>(n->y32, V, u);
    MGFR_HIP(hipGetLastError());
    MGFR_HIP(hipStreamSynchronize(n->stream));
    return MGFR_OK;
}

extern "C" int mgfr_net_activation(mgfr_net *n, int index, void *dst, int64_t count)
{
    if (!n || !dst) return set_error(MGFR_ERR_ARG, "net and dst must be non-NULL");
    if (index < 0 || index > 15) return set_error(MGFR_ERR_ARG, "activation index must be in [0, 15]");
    if (n->fwd_B == 0) return set_error(MGFR_ERR_ARG, "no forward pass has run on this network yet");
    // buffer, channels and pooling depth (0: S^3, 1: (S/2)^3, 2: (S/4)^3) in forward order
    // (the convolutions read a concatenation from its two sources: those are formed
    // here, in the scratch of the gradients)
    const __bf16 *buf[15] = {n->x0, n->h1a, n->s1, n->p1, n->h2a, n->s2, n->p2, n->h3a,
                             n->h3, n->gA, n->h4a, n->h4, n->gA, n->h5a, n->h5};
    static const int ch[16] = {16, 16, 16, 16, 32, 32, 32, 64, 64, 96, 32, 32, 48, 16, 16, 1};
    static const int depth[16] = {0, 0, 0, 1, 1, 1, 2, 2, 2, 1, 1, 1, 0, 0, 0, 0};
    const size_t vox = ((size_t)n->fwd_B << (3 * n->fwd_lg)) >> (3 * depth[index]);
    const size_t elems = vox * ch[index];
    if (count != (int64_t)elems) return set_error(MGFR_ERR_ARG, "count does not match the activation's size");
    if (index == 9)
        k_concat_up<<<gridn(vox * 12), 256, 0, n->stream>>>(n->h3, 64, n->s2, 32, n->fwd_lg - 1, vox, n->gA);
    if (index == 12)
        k_concat_up<<<gridn(vox * 6), 256, 0, n->stream>>>(n->h4, 32, n->s1, 16, n->fwd_lg, vox, n->gA);
    MGFR_HIP(hipGetLastError());
    const void *src = index == 15 ? (const void *)n->y32 : (const void *)buf[index];
    const size_t esz = index == 15 ? sizeof(float) : sizeof(__bf16);
    MGFR_HIP(hipMemcpyAsync(dst, src, elems * esz, hipMemcpyDeviceToDevice, n->stream));
    MGFR_HIP(hipStreamSynchronize(n->stream));
    return MGFR_OK;
}

extern "C" int mgfr_net_train_step(mgfr_net *n, const double *delta, const double *u_target, int B, int S,
                                   const double *cond, float lr, float *loss)
{
    if (!n || !delta || !u_target || !cond) return set_error(MGFR_ERR_ARG, "net, delta, u_target and cond must be non-NULL");
    if (!(lr > 0.f)) return set_error(MGFR_ERR_ARG, "lr must be > 0");
    int lgS, rc;
    if ((rc = check_shape(n, B, S, &lgS))) return rc;
    set_cond(n, cond, B);
    if ((rc = net_forward(n, delta, B, lgS))) return rc;
    if ((rc = net_backward(n, u_target, B, lgS))) return rc;
    n->step += 1;
    const float b1 = 0.9f, b2 = 0.999f;
    const float c1 = 1.f - std::pow(b1, (float)n->step), c2 = 1.f - std::pow(b2, (float)n->step);
    k_adam<<<gridn(n->nparam), 256, 0, n->stream>>>(n->p, n->g, n->m, n->v, n->nparam, lr, b1, b2, 1e-8f, c1, c2);
    if ((rc = net_refresh(n))) return rc;
    MGFR_HIP(hipMemcpyAsync(n->hloss, n->loss, sizeof(float), hipMemcpyDeviceToHost, n->stream));
    MGFR_HIP(hipStreamSynchronize(n->stream));
    if (loss) *loss = *n->hloss;
    if (!std::isfinite(*n->hloss)) return set_error(MGFR_ERR_NONFINITE, "training loss is not finite");
    return MGFR_OK;
}

extern "C" int mgfr_net_grads(mgfr_net *n, const double *delta, const double *u_target, int B, int S,
                              const double *cond, float *loss, float *grad_host)
{
    if (!n || !delta || !u_target || !cond || !grad_host) return set_error(MGFR_ERR_ARG, "null argument");
    int lgS, rc;
    if ((rc = check_shape(n, B, S, &lgS))) return rc;
    set_cond(n, cond, B);
    if ((rc = net_forward(n, delta, B, lgS))) return rc;
    if ((rc = net_backward(n, u_target, B, lgS))) return rc;
    MGFR_HIP(hipMemcpyAsync(grad_host, n->g, n->nparam * sizeof(float), hipMemcpyDeviceToHost, n->stream));
    MGFR_HIP(hipMemcpyAsync(n->hloss, n->loss, sizeof(float), hipMemcpyDeviceToHost, n->stream));
    MGFR_HIP(hipStreamSynchronize(n->stream));
    if (loss) *loss = *n->hloss;
    return MGFR_OK;
}

// ----------------------------------------------------- single-layer entry points

static int conv_args(int B, int S, int Cin, int Cout, int *lgS)
{
    if (B < 1 || S < 8 || (S & (S - 1))) return set_error(MGFR_ERR_ARG, "B >= 1 and power-of-two S >= 8 required");
    if (Cin < 8 || Cin % 8 || Cin > 96) return set_error(MGFR_ERR_ARG, "Cin must be a multiple of 8 in [8, 96]");
    if (Cout < 16 || Cout % 16 || Cout > 96) return set_error(MGFR_ERR_ARG, "Cout must be a multiple of 16 in [16, 96]");
    int lg = 0;
    while ((1 << lg) < S) ++lg;
    *lgS = lg;
    return MGFR_OK;
}

extern "C" int mgfr_conv3d_fwd(const void *x, int B, int S, int Cin, const void *w, const float *bias, int Cout,
                               int relu, void *y, float *y32, void *stream)
{
    int lgS, rc;
    if ((rc = conv_args(B, S, Cin, Cout, &lgS))) return rc;
    if (!x || !w || (!y && !y32)) return set_error(MGFR_ERR_ARG, "x, w and an output must be non-NULL");
    const size_t V = (size_t)B << (3 * lgS);
    return launch_conv3d({(const __bf16 *)x, Cin}, V, lgS, (const __bf16 *)w, bias, Cout, relu, nullptr, (__bf16 *)y, y32,
                         (hipStream_t)stream);
}

extern "C" int mgfr_conv3d_bwd_data(const void *dz, int B, int S, int Cout, const void *w, int Cin, void *wt_work,
                                    void *dx, void *stream)
{
    int lgS, rc;
    if ((rc = conv_args(B, S, Cout, Cin, &lgS))) return rc;
    if (Cin % 16 || Cout % 8) return set_error(MGFR_ERR_ARG, "backward-data needs Cin % 16 == 0");
    if (!dz || !w || !wt_work || !dx) return set_error(MGFR_ERR_ARG, "null argument");
    hipStream_t s = (hipStream_t)stream;
    k_wt_transpose<<<gridn((size_t)27 * Cin * Cout), 256, 0, s>>>((const __bf16 *)w, Cin, Cout, (__bf16 *)wt_work);
    const size_t V = (size_t)B << (3 * lgS);
    return launch_conv3d({(const __bf16 *)dz, Cout}, V, lgS, (const __bf16 *)wt_work, nullptr, Cin, 0, nullptr,
                         (__bf16 *)dx, nullptr, s);
}

extern "C" int mgfr_conv3d_bwd_weight(const void *x, const void *dz, int B, int S, int Cin, int Cout, float *dw,
                                      float *db, void *stream)
{
    int lgS, rc;
    if ((rc = conv_args(B, S, Cin, Cout, &lgS))) return rc;
    if (Cin % 16) return set_error(MGFR_ERR_ARG, "backward-weight needs Cin % 16 == 0");
    if (!x || !dz || !dw) return set_error(MGFR_ERR_ARG, "null argument");
    hipStream_t s = (hipStream_t)stream;
    const size_t V = (size_t)B << (3 * lgS);
    launch_wgrad({(const __bf16 *)x, Cin}, (const __bf16 *)dz, V, lgS, Cout, dw, db, s);
    MGFR_HIP(hipGetLastError());
    return MGFR_OK;
}

// ------------------------------------------------------------ solver hook

extern "C" int mgfr_set_net(mgfr_ctx *c, mgfr_net *n)
{
    if (!c) return set_error(MGFR_ERR_ARG, "ctx is NULL");
    nn_free(c);
    c->nn = n;
    return MGFR_OK;
}

// The context's own network (the mgfr_nn_* calls): capacity for the N/4 mesh
// and for training batches of eight 64^3 volumes.
extern "C" int mgfr_nn_init(mgfr_ctx *c, int seed)
{
    if (!c) return set_error(MGFR_ERR_ARG, "ctx is NULL");
    const int64_t n4 = (int64_t)(c->lev[0].N / 4) * (c->lev[0].N / 4) * (c->lev[0].N / 4);
    const int64_t cap = std::max<int64_t>({n4, (int64_t)8 * 64 * 64 * 64});
    mgfr_net *n = nullptr;
    int rc = mgfr_net_create(seed, (cap + 4095) / 4096 * 4096, c->stream, &n);
    if (rc) return rc;
    nn_free(c);
    c->nn = n;
    c->nn_owned = true;
    return MGFR_OK;
}

namespace {
mgfr_net *ctx_net(mgfr_ctx *c)
{
    if (!c) {
        set_error(MGFR_ERR_ARG, "ctx is NULL");
        return nullptr;
    }
    if (!c->nn) set_error(MGFR_ERR_ARG, "no network: call mgfr_nn_init or mgfr_set_net first");
    return (mgfr_net *)c->nn;
}
}  // namespace

extern "C" int mgfr_nn_train_step(mgfr_ctx *c, const double *delta, const double *u_target, int B, int S,
                                  const double *cond, float lr, float *loss)
{
    mgfr_net *n = ctx_net(c);
    if (!n) return MGFR_ERR_ARG;
    int rc = mgfr_net_set_stream(n, c->stream);
    return rc ? rc : mgfr_net_train_step(n, delta, u_target, B, S, cond, lr, loss);
}

extern "C" int mgfr_nn_predict(mgfr_ctx *c, const double *delta, double *u0)
{
    mgfr_net *n = ctx_net(c);
    if (!n) return MGFR_ERR_ARG;
    if (!delta || !u0) return set_error(MGFR_ERR_ARG, "delta and u0 must be non-NULL");
    const int cc = c->p.coarse_cycles;
    c->p.coarse_cycles = 0;  // the guess itself, without the coarse-level V-cycles of a solve
    double ms = 0.0;
    const int rc = nn_warm_start(c, delta, u0, &ms);
    c->p.coarse_cycles = cc;
    return rc;
}

extern "C" int mgfr_nn_save(mgfr_ctx *c, const char *path)
{
    mgfr_net *n = ctx_net(c);
    return n ? mgfr_net_save(n, path) : MGFR_ERR_ARG;
}

extern "C" int mgfr_nn_load(mgfr_ctx *c, const char *path)
{
    mgfr_net *n = ctx_net(c);
    return n ? mgfr_net_load(n, path) : MGFR_ERR_ARG;
}

namespace mgfr {

int nn_warm_start(mgfr_ctx *c, const double *delta, double *u, double *t_ms)
{
    mgfr_net *n = (mgfr_net *)c->nn;
    if (!n) return set_error(MGFR_ERR_ARG, "nn_mode needs a network attached with mgfr_set_net");
    if (c->nlev < 3 || c->lev[2].N < 32)
        return set_error(MGFR_ERR_ARG, "the network warm start needs N >= 128 (prediction on the N/4 mesh)");
    Level &L1 = c->lev[1], &L2 = c->lev[2];
    const int lg2 = L2.lg;
    const size_t n2 = (size_t)1 << (3 * lg2), n1 = (size_t)1 << (3 * L1.lg);
    if (n2 > n->maxvox) return set_error(MGFR_ERR_ARG, "the network's capacity is smaller than the N/4 mesh");
    hipStream_t saved = n->stream;
    n->stream = c->stream;
    MGFR_HIP(hipEventRecord(c->ev_c, c->stream));
    // delta on the N/4 mesh (means of 4^3 cells), network prediction of u there
    k_restrict4<<<gridn(n2), 256, 0, c->stream>>>(delta, lg2, L2.f);
    const double cond[2] = {c->p.a, c->p.fr0_abs};
    set_cond(n, cond, 1);
    int rc = net_forward(n, L2.f, 1, lg2);
    n->stream = saved;
    if (rc) return rc;
    k_to_u<<<gridn(n2), 256, 0, c->stream>>>(n->y32, n2, L2.u);
    // Coarse correction (nested iteration): the prediction is the initial guess
    // of the N/4 problem L(u) = R R f, which gets coarse_cycles V-cycles; its
    // solution, prolonged, starts coarse_cycles V-cycles of the N/2 problem
    // L(u) = R f, whose solution prolonged is the initial guess at N.  With
    // coarse_cycles = 0 the prediction is prolonged directly.
    const int cc = c->p.coarse_cycles;
    if (cc > 0) {
        k_restrict_mean<<<gridn(n1), 256, 0, c->stream>>>(c->lev[0].f, L1.lg, L1.f);
        k_restrict_mean<<<gridn(n2), 256, 0, c->stream>>>(L1.f, lg2, L2.f);
        MGFR_HIP(hipGetLastError());
        for (int k = 0; k < cc; ++k)
            if ((rc = vcycle64(c, 2))) return rc;
    }
    // prolong twice with the linear reconstruction (Sec. 3.3)
    k_prolong_field_set<<<(unsigned)((n2 + kBlock - 1) / kBlock), kBlock, 0, c->stream>>>(L1.u, L2.u, lg2);
    for (int k = 0; k < cc; ++k)
        if ((rc = vcycle64(c, 1))) return rc;
    k_prolong_field_set<<<(unsigned)((n1 + kBlock - 1) / kBlock), kBlock, 0, c->stream>>>(u, L1.u, L1.lg);
    MGFR_HIP(hipGetLastError());
    MGFR_HIP(hipEventRecord(c->ev_b, c->stream));
    MGFR_HIP(hipEventSynchronize(c->ev_b));
    float ms = 0.f;
    MGFR_HIP(hipEventElapsedTime(&ms, c->ev_c, c->ev_b));
    *t_ms = ms;
    return MGFR_OK;
}

// detach the network; destroy it if the context created it (mgfr_nn_init)
void nn_free(mgfr_ctx *c)
{
    if (c->nn_owned && c->nn) mgfr_net_destroy((mgfr_net *)c->nn);
    c->nn = nullptr;
    c->nn_owned = false;
}

}  // namespace mgfr
