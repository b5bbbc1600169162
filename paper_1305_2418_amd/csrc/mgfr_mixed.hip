// Mixed-precision solve: float64 defect correction around float32 FAS V-cycles.
//
// Outer loop (float64, finest level only):
//   r = f - L(u)                      residual of the float64 iterate
//   stop when max|r| / D <= tol       (Sec. 3.3 step 8)
//   solve N_u(e) = r approximately    one float32 FAS V-cycle, e = 0 initially
//   u <- u + e
// where N_u(e) = L(u + e) - L(u) is evaluated without cancellation:
//   N_c = (1/h^2) sum_nb [ (w_n X_n + w_c X_c)/2 (u_n - u_c)
//                          + (w_n (1 + X_n) + w_c (1 + X_c))/2 (e_n - e_c) ]
//         + bC s_c expm1(-q e_c)
// with w = e^u, s = e^{-q u}, X = expm1(e).  The float32 unknown is the small
// correction, so float32 keeps its relative precision and the float64
// residual can still reach 1e-8.  The inner cycle is the same FAS V-cycle as
// the float64 solve (Sec. 3.3): restriction by daughter means of e and of the
// linearisation point u, coarse source N_2h(R e) + R(r - N(e)), correction
// e += P(e_2h - R e), red-black Newton-Gauss-Seidel on e.  In exact
// arithmetic one such cycle from e = 0 reproduces one float64 V-cycle, so the
// float64 residual follows the float64 solve's history to rounding.  If it
// grows for three consecutive outer iterations (the float64 solve itself shows
// two-step transients from a cold start in deep screening) or turns
// non-finite, the solve restarts as the plain float64 solve from u = 0.
#include "mgfr_internal.h"
#include "mgfr_ops.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>

namespace mgfr {

namespace {


__device__ __forceinline__ size_t ix(int i, int j, int k, int lg)
{
    return (((((size_t)i) << lg) + (size_t)j) << lg) + (size_t)k;
}

// Index of cell (i,j,k) in a float32 correction-cycle array e, r or ebar of a
// level: natural order, or (split) every (i,j) row holding its cells with
// i + j + k even first (in k order), then the odd ones, so that a one-colour
// pass reads and writes its half of a row contiguously.  u32 is always natural.
__device__ __forceinline__ size_t sx(int i, int j, int k, int lg, bool split)
{
    const size_t row = ((((size_t)i) << lg) + (size_t)j) << lg;
    return split ? row + ((size_t)((i + j + k) & 1) << (lg - 1)) + (size_t)(k >> 1) : row + (size_t)k;
}

__device__ __forceinline__ double nanmax_d(double a, double b) { return (a != a || a > b) ? a : b; }

// gather the cell and its six periodic neighbours and their exponentials
struct MxCell {
    float ec, Xc, uc, wc;
    float en[6], Xn[6], un[6], wn[6];
};

__device__ __forceinline__ void mx_gather(const float *__restrict__ e, const float *__restrict__ u, int i, int j,
                                          int k, int lg, MxCell &c, bool split = false)
{
    const int m = (1 << lg) - 1;
    const int ni[6] = {(i + 1) & m, (i - 1) & m, i, i, i, i}, nj[6] = {j, j, (j + 1) & m, (j - 1) & m, j, j},
              nk[6] = {k, k, k, k, (k + 1) & m, (k - 1) & m};
    c.ec = e[sx(i, j, k, lg, split)];
    c.uc = u[ix(i, j, k, lg)];
    c.Xc = fexpm1(c.ec);
    c.wc = fexp(c.uc);
#pragma unroll
    for (int t = 0; t < 6; ++t) {
        c.en[t] = e[sx(ni[t], nj[t], nk[t], lg, split)];
        c.un[t] = u[ix(ni[t], nj[t], nk[t], lg)];
        c.Xn[t] = fexpm1(c.en[t]);
        c.wn[t] = fexp(c.un[t]);
    }
}

__device__ __forceinline__ void mx_sweep_cell(float *__restrict__ e, const float *__restrict__ u,
                                              const float *__restrict__ r, size_t t, int lg, int colour,
                                              const MxConst &kc)
{
    const int m = (1 << lg) - 1;
    const int mh = (int)(t & (size_t)((1 << (lg - 1)) - 1));
    const size_t row = t >> (lg - 1);
    const int j = (int)(row & m), i = (int)(row >> lg);
    const int k = 2 * mh + ((i + j + colour) & 1);
    MxCell c;
    mx_gather(e, u, i, j, k, lg, c);
    const size_t cc = ix(i, j, k, lg);
    e[cc] = c.ec + mx_step(c.ec, c.Xc, c.uc, c.wc, c.en, c.Xn, c.un, c.wn, r[cc], kc);
}

__device__ __forceinline__ float mx_value_at(const float *__restrict__ e, const float *__restrict__ u, int i, int j,
                                             int k, int lg, const MxConst &kc, bool split = false)
{
    MxCell c;
    mx_gather(e, u, i, j, k, lg, c, split);
    return mx_value(c.ec, c.Xc, c.uc, c.wc, c.en, c.Xn, c.un, c.wn, kc);
}

// Daughter means of e, u and of the residual r - N(e) for coarse cell (I,J,K):
// the 2x2x2 block and its 24 face neighbours are loaded and exponentiated once.
__device__ __forceinline__ void mx_restrict_block(const float *__restrict__ e, const float *__restrict__ u,
                                                  const float *__restrict__ r, int I, int J, int K, int lg,
                                                  const MxConst &kc, float &em, float &um, float &rm, bool split)
{
    const int m = (1 << lg) - 1;
    const int i0 = 2 * I, j0 = 2 * J, k0 = 2 * K;
    // index 0..7: block cell (a,b,c) -> a*4+b*2+c; faces: [face][p][q]
    float Be[8], Bu[8], BX[8], Bw[8];
    float Fe[6][4], Fu[6][4], FX[6][4], Fw[6][4];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                Be[a * 4 + b * 2 + c] = e[sx(i0 + a, j0 + b, k0 + c, lg, split)];
                Bu[a * 4 + b * 2 + c] = u[ix(i0 + a, j0 + b, k0 + c, lg)];
            }
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int fi[6] = {(i0 + 2) & m, (i0 - 1) & m, i0 + p, i0 + p, i0 + p, i0 + p};
            const int fj[6] = {j0 + p, j0 + p, (j0 + 2) & m, (j0 - 1) & m, j0 + q, j0 + q};
            const int fk[6] = {k0 + q, k0 + q, k0 + q, k0 + q, (k0 + 2) & m, (k0 - 1) & m};
#pragma unroll
            for (int f = 0; f < 6; ++f) {
                Fe[f][p * 2 + q] = e[sx(fi[f], fj[f], fk[f], lg, split)];
                Fu[f][p * 2 + q] = u[ix(fi[f], fj[f], fk[f], lg)];
            }
        }
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        BX[t] = fexpm1(Be[t]);
        Bw[t] = fexp(Bu[t]);
    }
#pragma unroll
    for (int f = 0; f < 6; ++f)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            FX[f][t] = fexpm1(Fe[f][t]);
            Fw[f][t] = fexp(Fu[f][t]);
        }
    float se = 0.f, su = 0.f, sr = 0.f;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int t = a * 4 + b * 2 + c;
                // neighbours +x, -x, +y, -y, +z, -z: inside the block or on a face
                const int nx0 = (a ^ 1) * 4 + b * 2 + c;
                const int ny0 = a * 4 + (b ^ 1) * 2 + c;
                const int nz0 = a * 4 + b * 2 + (c ^ 1);
                float en[6], Xn[6], un[6], wn[6];
#define MX_NB(slot, inblock, bi, face, fi)                                                  \
    if (inblock) { en[slot] = Be[bi]; Xn[slot] = BX[bi]; un[slot] = Bu[bi]; wn[slot] = Bw[bi]; } \
    else { en[slot] = Fe[face][fi]; Xn[slot] = FX[face][fi]; un[slot] = Fu[face][fi]; wn[slot] = Fw[face][fi]; }
                MX_NB(0, a == 0, nx0, 0, b * 2 + c)
                MX_NB(1, a == 1, nx0, 1, b * 2 + c)
                MX_NB(2, b == 0, ny0, 2, a * 2 + c)
                MX_NB(3, b == 1, ny0, 3, a * 2 + c)
                MX_NB(4, c == 0, nz0, 4, a * 2 + b)
                MX_NB(5, c == 1, nz0, 5, a * 2 + b)
#undef MX_NB
                const float N = mx_value(Be[t], BX[t], Bu[t], Bw[t], en, Xn, un, wn, kc);
                se += Be[t];
                su += Bu[t];
                sr += r[sx(i0 + a, j0 + b, k0 + c, lg, split)] - N;
            }
    em = 0.125f * se;
    um = 0.125f * su;
    rm = 0.125f * sr;
}

// Element at a wave-uniform row pointer plus a 32-bit byte offset (lets the
// compiler address with a scalar base and one 32-bit lane offset).
template <typename T>
__device__ __forceinline__ const T &at_off(const float *base, uint32_t byte_off)
{
    return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) + byte_off);
}
template <typename T>
__device__ __forceinline__ T &at_off(float *base, uint32_t byte_off)
{
    return *reinterpret_cast<T *>(reinterpret_cast<char *>(base) + byte_off);
}

// ---------------------------------------------------------- colour pass (N >= 128)
//
// One colour of the float32 correction sweep on a level with N >= 128: the
// cells with (i + j + k) & 1 == colour are updated in place; all six
// neighbours of such a cell have the other colour and are only read.
// Workgroup: CTJ rows of a 128-cell row tile plus one halo row on each side,
// one wave per row, marching over `chunk` planes.  Lane l holds the pair
// k = k0 + 2l, k0 + 2l + 1 of its row; in each plane one of the two is updated
// (column s, the same for the whole wave) and the other is published in LDS
// for the rows above and below and the neighbouring lanes.  s alternates from
// plane to plane, so the plane loop is written out for both parities.  e^u and
// expm1(e) of a cell are evaluated once, when its plane is loaded, and kept as
// P = e^u expm1(e) and W = e^(u+e); the cells beyond the tile's ends in k come
// from the first lanes of the upper halo wave.
// e, r and ebar of such a level are stored split by colour (see sx), so the
// pass reads r and writes e of its half only: 12 B per cell.

#ifndef MGFR_CTJ
#define MGFR_CTJ 8
#endif
constexpr int CTJ = MGFR_CTJ;  // updated rows per workgroup (the last row tile may be partial)
#ifndef MGFR_COLOUR_PF
#define MGFR_COLOUR_PF 3
#endif
constexpr int kColourPf = MGFR_COLOUR_PF;  // planes between a raw load and its use (1, 2 or 3)
static_assert(kColourPf >= 1 && kColourPf <= 3, "prefetch distance 1, 2 or 3");
// Planes per workgroup (a multiple of 4): N / 8, but 8 at 128^3, where N / 8
// leaves half the CUs without a workgroup.  us per pass with 8, 16, 32 chunks:
// 128^3 12.5, 8.6, 10.5; 256^3 45, 49, 59; 512^3 389, 425, 463 (each chunk's
// start costs).
inline int colour_chunk(int N) { return N <= 128 ? 8 : N / 8; }
constexpr int CKW = 128;  // cells per row tile
constexpr int CLW = 66;   // LDS row: 64 lanes and one halo slot on each side

struct Cell4 {
    float u, e, P, W;
};

__device__ __forceinline__ Cell4 mx_cell(float u, float e)
{
    const float w = fexp(u);
    const float P = w * fexpm1(e);
    return Cell4{u, e, P, w + P};
}

__device__ __forceinline__ float4 pack(const Cell4 &c) { return make_float4(c.u, c.e, c.P, c.W); }
__device__ __forceinline__ Cell4 unpack(const float4 &v) { return Cell4{v.x, v.y, v.z, v.w}; }

// c ? a : b, value by value (a select of two objects would put them in scratch memory)
__device__ __forceinline__ Cell4 sel(bool c, const Cell4 &a, const Cell4 &b)
{
    return Cell4{c ? a.u : b.u, c ? a.e : b.e, c ? a.P : b.P, c ? a.W : b.W};
}

// New e at a cell from the cell, its residual target r and its six neighbours
// (the same Newton step as mx_step, on the P/W form).
__device__ __forceinline__ float mx_update(const Cell4 &c, float r, const Cell4 &n0, const Cell4 &n1,
                                           const Cell4 &n2, const Cell4 &n3, const Cell4 &n4, const Cell4 &n5,
                                           const MxConst &k)
{
    float Su = n0.u - c.u, Se = n0.e - c.e;
    float A = n0.P * Su, B = n0.W * Se, SW = n0.W;
    auto add = [&](const Cell4 &n) {
        const float du = n.u - c.u, de = n.e - c.e;
        Su += du;
        Se += de;
        A = fmaf(n.P, du, A);
        B = fmaf(n.W, de, B);
        SW += n.W;
    };
    add(n1);
    add(n2);
    add(n3);
    add(n4);
    add(n5);
    // twice the flux and its derivative; ih2h = 1 / (2 h^2) (halving is exact)
    const float ih2h = 0.5f * k.ih2;
    const float flux2 = fmaf(c.P, Su, A) + fmaf(c.W, Se, B);
    const float dflux2 = fmaf(c.W, Su + Se - 6.0f, -SW);
    const float sc = fexp(-k.q * c.u);
    const float cm = fexpm1(-k.q * c.e);
    const float N = fmaf(k.bC * sc, cm, ih2h * flux2);
    const float J = fmaf(ih2h, dflux2, -(k.q * k.bC * sc * (1.0f + cm)));
    float d = -(N - r) * __builtin_amdgcn_rcpf(J) * k.omega;
    if (k.max_du > 0.f) d = fminf(fmaxf(d, -k.max_du), k.max_du);
    return c.e + d;
}

struct ColourArgs {
    float *e;
    const float *u, *r;
    int lg, colour, chunk;
    MxConst kc;
};

// The plane loop of one wave whose updated column in the first plane is S0.
// ZERO: e is zero everywhere (the first pass of a correction cycle): nothing
// of e is read, and the cells of the other colour are written as 0, so that
// the array need not be cleared beforehand.
template <int S0, bool ZERO>
__device__ __forceinline__ void mx_colour_rows(const ColourArgs &A, int i0, int j0, int k0, int wv, int lane,
                                               float4 *sB)
{
    const int lg = A.lg, m = (1 << lg) - 1;
    const size_t hN = (size_t)1 << (lg - 1);
    const int row = wv - 1;                      // -1 and CTJ: halo rows
    const bool upd = row >= 0 && row < CTJ && j0 + row <= m;  // uniform over the wave
    const int jg = (j0 + row) & m;
    const size_t plane = (size_t)1 << (2 * lg);
    const size_t rowbase = (size_t)jg << lg;
    // rows that update nothing load r of the tile's first row (already fetched)
    const size_t rrowbase = upd ? rowbase : (size_t)j0 << lg;
    // addresses: a wave-uniform row pointer (scalar arithmetic) plus a 32-bit lane offset
    const uint32_t kk = 4u * (uint32_t)(k0 + 2 * lane), kh2 = 4u * (uint32_t)(k0 / 2 + lane);  // byte offsets
    auto pb = [&](int pl) { return (size_t)(pl & m) * plane + rowbase; };
    // u in natural order; e and r split by colour (column 0 of plane pl lies in half (pl + jg) & 1)
    auto ldu = [&](int pl) { return at_off<float2>(A.u + pb(pl), kk); };
    auto lde = [&](int pl) {
        if constexpr (ZERO) return make_float2(0.0f, 0.0f);
        const bool odd = ((pl + jg) & 1) != 0;
        const float *h0 = A.e + pb(pl) + (odd ? hN : 0), *h1 = A.e + pb(pl) + (odd ? 0 : hN);
        return make_float2(at_off<float>(h0, kh2), at_off<float>(h1, kh2));
    };
    auto row_c = [&](int pl) { return A.e + pb(pl) + (size_t)A.colour * hN; };  // half of the updated cells
    auto row_r = [&](int pl) { return A.r + (size_t)(pl & m) * plane + rrowbase + (size_t)A.colour * hN; };
    // k-halo duty: lanes 0..CTJ-1 of the upper halo wave serve row `lane`.  Every
    // lane of every wave issues the same loads in every plane (lane mod CTJ), so
    // that no load sits under a branch and the prefetch waits stay exact.
    const bool kh = wv == 0 && lane < CTJ;
    const int khq = lane % CTJ;
    const size_t khrow = (size_t)((j0 + khq) & m) << lg;
    const int khpar = (A.colour + j0 + khq) & 1;  // updated column of that row in even planes
    auto kh_k = [&](int pl) { return (khpar ^ (pl & 1)) ? ((k0 + CKW) & m) : ((k0 - 1) & m); };
    auto kh_u = [&](int pl) { return (size_t)(pl & m) * plane + khrow + (size_t)kh_k(pl); };
    // the halo cell has the other colour
    auto kh_e = [&](int pl) {
        return (size_t)(pl & m) * plane + khrow + (size_t)(1 - A.colour) * hN + (size_t)(kh_k(pl) >> 1);
    };
    auto kh_slot = [&](int pl) { return (lane + 1) * CLW + ((khpar ^ (pl & 1)) ? CLW - 1 : 0); };

    // prologue: plane i0 (both columns), plane i0 - 1 (column S0), raw plane i0 + 1
    Cell4 c0, c1, prev;
    {
        const float2 u0 = ldu(i0), e0 = lde(i0);
        const float2 um = ldu(i0 - 1), em = lde(i0 - 1);
        c0 = mx_cell(u0.x, e0.x);
        c1 = mx_cell(u0.y, e0.y);
        prev = S0 ? mx_cell(um.y, em.y) : mx_cell(um.x, em.x);
    }
    // raw loads of step p: u, e of plane p + 1, r of plane p, the k-halo cell of plane p.
    // They are issued kColourPf steps ahead; four register sets rotate with the
    // four-plane loop body, so that no register holding a load in flight is copied.
    struct Raw {
        float2 u, e;
        float r, khu, khe;
    };
    auto load = [&](int p) {
        Raw w;
        w.u = ldu(p + 1);
        w.e = lde(p + 1);
        w.r = at_off<float>(row_r(p), kh2);
        w.khu = A.u[kh_u(p)];
        w.khe = ZERO ? 0.0f : A.e[kh_e(p)];
        return w;
    };
    Raw ra = load(i0), rb = kColourPf >= 2 ? load(i0 + 1) : Raw{}, rc = kColourPf == 3 ? load(i0 + 2) : Raw{}, rd;
    int buf = 0;

    // one plane with updated column S: consume cur (step p), load nxt (step p + kColourPf)
    auto step = [&](int p, auto Sc, const Raw &cur, Raw &nxt) {
        constexpr int S = decltype(Sc)::value;
        nxt = load(p + kColourPf);
        // plane p + 1 from the raw values loaded kColourPf planes ago
        const Cell4 n0 = mx_cell(cur.u.x, cur.e.x), n1 = mx_cell(cur.u.y, cur.e.y);
        float4 *B = sB + buf * (CTJ + 2) * CLW;
        B[(row + 1) * CLW + lane + 1] = pack(S ? c0 : c1);
        if (kh) B[kh_slot(p)] = pack(mx_cell(cur.khu, cur.khe));
        __syncthreads();
        if (upd) {
            const Cell4 up = unpack(B[row * CLW + lane + 1]);
            const Cell4 dn = unpack(B[(row + 2) * CLW + lane + 1]);
            const Cell4 sd = unpack(B[(row + 1) * CLW + lane + (S ? 2 : 0)]);
            const float en = S ? mx_update(c1, cur.r, c0, sd, up, dn, prev, n1, A.kc)
                               : mx_update(c0, cur.r, c1, sd, up, dn, prev, n0, A.kc);
            at_off<float>(row_c(p), kh2) = en;
            if constexpr (ZERO) at_off<float>(A.e + pb(p) + (size_t)(1 - A.colour) * hN, kh2) = 0.0f;
        }
        prev = S ? c0 : c1;
        c0 = n0;
        c1 = n1;
        buf ^= 1;
    };
    using Z0 = std::integral_constant<int, S0>;
    using Z1 = std::integral_constant<int, 1 - S0>;
    if constexpr (kColourPf == 3) {
        for (int p = i0; p < i0 + A.chunk; p += 4) {  // chunk is a multiple of 4
            step(p, Z0{}, ra, rd);
            step(p + 1, Z1{}, rb, ra);
            step(p + 2, Z0{}, rc, rb);
            step(p + 3, Z1{}, rd, rc);
        }
    } else if constexpr (kColourPf == 2) {
        for (int p = i0; p < i0 + A.chunk; p += 4) {
            step(p, Z0{}, ra, rc);
            step(p + 1, Z1{}, rb, rd);
            step(p + 2, Z0{}, rc, ra);
            step(p + 3, Z1{}, rd, rb);
        }
    } else {
        for (int p = i0; p < i0 + A.chunk; p += 2) {
            step(p, Z0{}, ra, rb);
            step(p + 1, Z1{}, rb, ra);
        }
    }
}

// grid: 1-D, (N / CKW) ceil(N / CTJ) (N / chunk) workgroups, spread so that
// workgroups adjacent in j run on the same XCD (they share halo rows)
template <bool ZERO>
__device__ __forceinline__ void mx_colour_pass(const ColourArgs &A, float4 *sB)
{
    const int lg = A.lg;
    const unsigned nb = gridDim.x, b = blockIdx.x;
    const unsigned L = (b & 7u) * (nb >> 3) + (b >> 3);  // nb is a multiple of 8
    const int nkt = (1 << lg) / CKW, njt = ((1 << lg) + CTJ - 1) / CTJ;
    const int kt = (int)(L % (unsigned)nkt), jt = (int)((L / (unsigned)nkt) % (unsigned)njt),
              it = (int)(L / ((unsigned)nkt * (unsigned)njt));
    const int k0 = kt * CKW, j0 = jt * CTJ, i0 = it * A.chunk;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    const int s0 = (A.colour + i0 + j0 + wv - 1) & 1;  // updated column of this wave's row in plane i0
    if (s0)
        mx_colour_rows<1, ZERO>(A, i0, j0, k0, wv, lane, sB);
    else
        mx_colour_rows<0, ZERO>(A, i0, j0, k0, wv, lane, sB);
}

__global__ __launch_bounds__(64 * (CTJ + 2)) void k_mx_colour(ColourArgs A)
{
    __shared__ float4 sB[2 * (CTJ + 2) * CLW];
    mx_colour_pass<false>(A, sB);
}

// the first pass of a correction cycle, from e = 0
__global__ __launch_bounds__(64 * (CTJ + 2)) void k_mx_colour_zero(ColourArgs A)
{
    __shared__ float4 sB[2 * (CTJ + 2) * CLW];
    mx_colour_pass<true>(A, sB);
}

// ------------------------------------------- fused red-black sweep (N >= 256)
//
// One whole float32 correction sweep (red cells, then black cells) in one
// launch, out of place: eout = sweep(ein) on a split level (see sx); the
// scheme of the float64 k_sweep_rows.  A workgroup has 15 waves, one per row
// of 128 cells (lane l: the pair k0 + 2 l, k0 + 2 l + 1), and marches along i; in
// step p it updates the red cells of plane p + 1 and the black cells of plane
// p - 1, two independent updates per lane.  Rows 1..13 are stored; rows 0 and
// 14 update only the red cells that rows 1 and 13 need.  A sixteenth wave
// updates the red cells k0 - 1 and k0 + 128 of all rows.  LDS holds the old
// black cells of plane p + 1 and the new red cells of plane p - 1 as
// (u, e, P, W).  The updates are those of the colour pass, operand by operand,
// so the iterates are the same bit for bit.
//
// Bound: vector issue (a SIMD's four waves fill a step) and, with one
// workgroup per CU, what a step cannot overlap; 16 B per cell of traffic
// instead of the two passes' 24.  512^3: 565 us per sweep against 730 us in
// two passes; updating the black cells of plane p after the red ones of plane
// p + 1, one after the other, took 910 us.
struct SweepRowsArgs {
    const float *ein;
    float *eout;
    const float *u, *r;
    int lg, chunk;
    unsigned nkt, njt;
    MxConst kc;
};

typedef float4 MxRowLds[2][kRowF][kRowS];

// S0: red column of the wave's row on plane i0 - 1.  RING: an outer row.  ZERO:
// e is zero everywhere and not read.
template <int S0, bool RING, bool ZERO>
__device__ __forceinline__ void mx_sweep_rows(const SweepRowsArgs &A, int i0, int j0, int k0, int row, int lane,
                                              MxRowLds &sO, MxRowLds &sN)
{
    const int lg = A.lg, m = (1 << lg) - 1;
    const int i1 = min(i0 + A.chunk, m + 1);
    const size_t plane = (size_t)1 << (2 * lg);
    const uint32_t pbytes = 4u << (2 * lg), hN = 2u << lg;  // bytes of a plane, of half a row
    const int jg = (j0 - 1 + row) & m;
    const bool stored = !RING && j0 - 1 + row <= m;  // uniform over the wave
    const uint32_t jo = (uint32_t)((row == 0 ? jg - 1 : jg + 1) & m) << lg;  // RING: the row beyond
    // byte offsets within a plane: the pair in natural order, its cells in a half row
    const uint32_t kk = (uint32_t)(k0 + 2 * lane);
    const uint32_t offu = 4u * (((uint32_t)jg << lg) + kk), offe = 4u * (((uint32_t)jg << lg) + (kk >> 1));
    const uint32_t offou = 4u * (jo + kk), offoe = 4u * (jo + (kk >> 1)) + hN;
    auto pu = [&](int pl) { return PlaneBuf(A.u + (size_t)(pl & m) * plane, pbytes); };
    auto pe = [&](int pl) { return PlaneBuf(A.ein + (size_t)(pl & m) * plane, pbytes); };
    auto pr = [&](int pl) { return PlaneBuf(A.r + (size_t)(pl & m) * plane, pbytes); };
    const MxConst &kc = A.kc;
    // raw values of step p, two steps ahead: u and e (red and black half) of plane
    // p + 2, r of the red cell of plane p + 1 and of the black cell of plane p - 1;
    // RING: the red cell's outer neighbour on plane p + 1 (a black cell)
    struct Raw {
        float2 u;
        float er, eb, rr, rb, ou, oe;
    };
    auto load = [&](int p, int S) {
        Raw w;
        w.u = pu(p + 2).ldf2(offu);
        w.er = w.eb = w.oe = 0.0f;
        if constexpr (!ZERO) {
            const PlaneBuf b = pe(p + 2);
            w.er = b.ldf(offe);
            w.eb = b.ldf(offe + hN);
        }
        w.rr = pr(p + 1).ldf(offe);
        if constexpr (RING) {
            w.ou = pu(p + 1).ldf(offou + 4u * S);
            if constexpr (!ZERO) w.oe = pe(p + 1).ldf(offoe);
        } else {
            w.rb = pr(p - 1).ldf(offe + hN);
        }
        return w;
    };
    // Planes p - 1 (red new), p (red new), p + 1 (old) and p + 2 of the pair in a
    // ring of four: the plane loop is written out for its four positions (and
    // both parities), so that no cell is moved between registers.
    Cell4 X[4][2];
    {
        // columns of plane i0 - 1: red S0; of plane i0 - 2: red 1 - S0
        const float2 u0 = pu(i0 - 2).ldf2(offu), u1 = pu(i0 - 1).ldf2(offu);
        float e0r = 0.f, e0b = 0.f, e1r = 0.f, e1b = 0.f;
        if constexpr (!ZERO) {
            e0r = pe(i0 - 2).ldf(offe);
            e0b = pe(i0 - 2).ldf(offe + hN);
            e1r = pe(i0 - 1).ldf(offe);
            e1b = pe(i0 - 1).ldf(offe + hN);
        }
        X[1][0] = mx_cell(u0.x, S0 ? e0r : e0b);
        X[1][1] = mx_cell(u0.y, S0 ? e0b : e0r);
        X[2][0] = mx_cell(u1.x, S0 ? e1b : e1r);
        X[2][1] = mx_cell(u1.y, S0 ? e1r : e1b);
        X[0][0] = X[0][1] = X[3][0] = X[3][1] = X[1][0];
    }
    Raw ra = load(i0 - 2, S0), rb = load(i0 - 1, 1 - S0);
    auto step = [&](int p, auto Hc, Raw &raw) {
        constexpr int H = decltype(Hc)::value, S = S0 ^ (H & 1), T = 1 - S;
        Cell4(&A1)[2] = X[H], (&C0)[2] = X[(H + 1) & 3], (&C1)[2] = X[(H + 2) & 3], (&Q)[2] = X[(H + 3) & 3];
        float4(*O)[kRowS] = sO[H & 1], (*R)[kRowS] = sN[H & 1];
        O[row][lane + 1] = pack(C1[T]);
        R[row][lane + 1] = pack(A1[S]);
        __syncthreads();
        const Cell4 R2 = Q[T];  // red cell of plane p - 2 (the ring's oldest plane)
        // plane p + 2: red column T
        Q[0] = mx_cell(raw.u.x, T ? raw.eb : raw.er);
        Q[1] = mx_cell(raw.u.y, T ? raw.er : raw.eb);
        const Raw cur = raw;
        raw = load(p + 2, S);
        // red cell of plane p + 1
        Cell4 up, dn;
        if constexpr (RING) {
            const Cell4 o = mx_cell(cur.ou, cur.oe), in = unpack(O[row == 0 ? 1 : row - 1][lane + 1]);
            up = sel(row == 0, o, in);
            dn = sel(row == 0, in, o);
        } else {
            up = unpack(O[row - 1][lane + 1]);
            dn = unpack(O[row + 1][lane + 1]);
        }
        const Cell4 sd = unpack(O[row][S ? lane + 2 : lane]);
        const float en = mx_update(C1[S], cur.rr, C1[T], sd, up, dn, C0[S], Q[S], kc);
        // black cell of plane p - 1
        if constexpr (!RING) {
            if (stored && p - 1 >= i0) {
                const Cell4 bu = unpack(R[row - 1][lane + 1]), bd = unpack(R[row + 1][lane + 1]),
                            bs = unpack(R[row][T ? lane + 2 : lane]);
                const PlaneBuf out(A.eout + (size_t)(p - 1) * plane, pbytes);
                out.stf(offe + hN, mx_update(A1[T], cur.rb, A1[S], bs, bu, bd, R2, C0[T], kc));
                out.stf(offe, A1[S].e);
            }
        }
        C1[S] = mx_cell(C1[S].u, en);
    };
    for (int p = i0 - 2;;) {
        step(p, std::integral_constant<int, 0>{}, ra);
        if (++p > i1) break;
        step(p, std::integral_constant<int, 1>{}, rb);
        if (++p > i1) break;
        step(p, std::integral_constant<int, 2>{}, ra);
        if (++p > i1) break;
        step(p, std::integral_constant<int, 3>{}, rb);
        if (++p > i1) break;
    }
}

// The red cells k0 - 1 (lanes 0..14, row = lane) and k0 + 128 (lanes 16..30) of
// the workgroup's rows, on the same steps: a cell is black and red in turn along
// i; black, its old value is published beside its row's black cells, red, it is
// updated and its new value published with the row's red ones.
template <bool ZERO>
__device__ __forceinline__ void mx_sweep_ends(const SweepRowsArgs &A, int i0, int j0, int k0, int lane, MxRowLds &sO,
                                              MxRowLds &sN)
{
    const int lg = A.lg, m = (1 << lg) - 1;
    const int i1 = min(i0 + A.chunk, m + 1);
    const size_t plane = (size_t)1 << (2 * lg);
    const uint32_t pbytes = 4u << (2 * lg), hN = 2u << lg;
    const bool low = (lane & 16) == 0, live = (lane & 15) < kRowF && lane < 32;
    const int q = min(lane & 15, kRowF - 1), slot = low ? 0 : kRowS - 1, in = low ? 1 : kRowS - 2;
    const int j = (j0 - 1 + q) & m, k = (low ? k0 - 1 : k0 + kRowW) & m, k2 = (low ? k0 - 2 : k0 + kRowW + 1) & m;
    const uint32_t row = (uint32_t)j << lg;
    // byte offsets within a plane: u and e of the cell and of its outer neighbour
    const uint32_t ou = 4u * (row + (uint32_t)k), oe = 4u * (row + (uint32_t)(k >> 1)), ou2 = 4u * (row + (uint32_t)k2),
                   oe2 = 4u * (row + (uint32_t)(k2 >> 1)) + hN;
    const int jup = q > 0 ? q - 1 : 0, jdn = q < kRowF - 1 ? q + 1 : q;
    auto pu = [&](int pl) { return PlaneBuf(A.u + (size_t)(pl & m) * plane, pbytes); };
    auto pe = [&](int pl) { return PlaneBuf(A.ein + (size_t)(pl & m) * plane, pbytes); };
    auto pr = [&](int pl) { return PlaneBuf(A.r + (size_t)(pl & m) * plane, pbytes); };
    auto lde = [&](int pl) { return ZERO ? 0.0f : pe(pl).ldf(oe + (((pl + j + k) & 1) ? hN : 0u)); };
    // step p: u, e of plane p + 2; r and the outer neighbour (black where the cell is red) of plane p + 1
    struct Raw {
        float u, e, r, u2, e2;
    };
    auto load = [&](int p) {
        Raw w;
        w.u = pu(p + 2).ldf(ou);
        w.e = lde(p + 2);
        w.r = pr(p + 1).ldf(oe);
        w.u2 = pu(p + 1).ldf(ou2);
        w.e2 = ZERO ? 0.0f : pe(p + 1).ldf(oe2);
        return w;
    };
    Cell4 X[4];  // planes p - 1, p, p + 1, p + 2 (ring)
    X[0] = X[1] = X[3] = mx_cell(pu(i0 - 2).ldf(ou), lde(i0 - 2));
    X[2] = mx_cell(pu(i0 - 1).ldf(ou), lde(i0 - 1));
    Raw ra = load(i0 - 2), rb = load(i0 - 1);
    auto step = [&](int p, auto Hc, Raw &raw) {
        constexpr int H = decltype(Hc)::value;
        const bool red = ((p + 1 + j + k) & 1) == 0;  // on planes p + 1 and p - 1
        float4(*O)[kRowS] = sO[H & 1], (*R)[kRowS] = sN[H & 1];
        if (live) (red ? R : O)[q][slot] = pack(sel(red, X[H], X[(H + 2) & 3]));
        __syncthreads();
        Cell4 &c = X[(H + 2) & 3], &n = X[(H + 3) & 3];
        n = mx_cell(raw.u, raw.e);
        const Raw cur = raw;
        raw = load(p + 2);
        if (live && red)
            c = mx_cell(c.u, mx_update(c, cur.r, mx_cell(cur.u2, cur.e2), unpack(O[q][in]), unpack(O[jup][slot]),
                                       unpack(O[jdn][slot]), X[(H + 1) & 3], n, A.kc));
    };
    for (int p = i0 - 2;;) {
        step(p, std::integral_constant<int, 0>{}, ra);
        if (++p > i1) break;
        step(p, std::integral_constant<int, 1>{}, rb);
        if (++p > i1) break;
        step(p, std::integral_constant<int, 2>{}, ra);
        if (++p > i1) break;
        step(p, std::integral_constant<int, 3>{}, rb);
        if (++p > i1) break;
    }
}

// grid: nkt njt ceil(N / chunk) workgroups; those of one XCD (blocks b, b + 8,
// ...) take consecutive tiles, which share their outer rows in its L2
template <bool ZERO>
__global__ __launch_bounds__(64 * (kRowF + 1)) void k_mx_sweep_rows(SweepRowsArgs A)
{
    __shared__ MxRowLds sO, sN;
    const unsigned nb = gridDim.x, x = blockIdx.x & 7u, per = nb >> 3, rem = nb & 7u;
    const unsigned L = x * per + min(x, rem) + (blockIdx.x >> 3);
    const int kt = (int)(L % A.nkt), jt = (int)((L / A.nkt) % A.njt), it = (int)(L / (A.nkt * A.njt));
    const int k0 = kt * kRowW, j0 = jt * kRowI, i0 = it * A.chunk;
    const int row = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    const int s0 = (i0 - 1 + j0 - 1 + row) & 1;  // red column of the row on plane i0 - 1
    if (row == kRowF)
        mx_sweep_ends<ZERO>(A, i0, j0, k0, lane, sO, sN);
    else if (row == 0 || row == kRowF - 1) {
        if (s0)
            mx_sweep_rows<1, true, ZERO>(A, i0, j0, k0, row, lane, sO, sN);
        else
            mx_sweep_rows<0, true, ZERO>(A, i0, j0, k0, row, lane, sO, sN);
    } else {
        if (s0)
            mx_sweep_rows<1, false, ZERO>(A, i0, j0, k0, row, lane, sO, sN);
        else
            mx_sweep_rows<0, false, ZERO>(A, i0, j0, k0, row, lane, sO, sN);
    }
}

// ------------------------------------------------- restriction pass (N >= 128)
//
// Residual restriction from a split level with N >= 128 to the next coarser
// level: for every coarse cell the means of e, u and r - N(e) over its eight
// daughters.  Same workgroups and plane march as the colour pass, but both
// cells of a lane's pair need N(e), so both are published in LDS and the
// k-halo holds both ends of every row.  The daughter sums run over the pair
// (lane), the row pair (adjacent waves, combined in LDS) and the plane pair
// (two consecutive steps).

__device__ __forceinline__ float mx_nval(const Cell4 &c, const Cell4 &n0, const Cell4 &n1, const Cell4 &n2,
                                         const Cell4 &n3, const Cell4 &n4, const Cell4 &n5, const MxConst &k)
{
    float Su = 0.f, Se = 0.f, A = 0.f, B = 0.f;
    auto add = [&](const Cell4 &n) {
        const float du = n.u - c.u, de = n.e - c.e;
        Su += du;
        Se += de;
        A = fmaf(n.P, du, A);
        B = fmaf(n.W, de, B);
    };
    add(n0);
    add(n1);
    add(n2);
    add(n3);
    add(n4);
    add(n5);
    const float flux = 0.5f * ((A + c.P * Su) + (B + c.W * Se));
    return k.ih2 * flux + k.bC * fexp(-k.q * c.u) * fexpm1(-k.q * c.e);
}

constexpr int PTJ = 8;  // fine rows per workgroup (even: rows pair up)

struct RestrictArgs {
    const float *e, *u, *r;
    float *ebc, *uc, *rc;
    int lg, chunk;
    bool split_c;
    MxConst kc;
};

__global__ __launch_bounds__(64 * (PTJ + 2)) void k_mx_restrict_pass(RestrictArgs A)
{
    __shared__ float4 sB[2 * (PTJ + 2) * CLW * 2];  // [buffer][row][slot][column]
    __shared__ float4 sR[PTJ / 2][64];               // odd rows' daughter sums
    const int lg = A.lg, m = (1 << lg) - 1, lgc = lg - 1;
    const size_t hN = (size_t)1 << (lg - 1);
    const unsigned nb = gridDim.x, b = blockIdx.x;
    const unsigned L = (b & 7u) * (nb >> 3) + (b >> 3);
    const int nkt = (1 << lg) / CKW, njt = (1 << lg) / PTJ;
    const int kt = (int)(L % (unsigned)nkt), jt = (int)((L / (unsigned)nkt) % (unsigned)njt),
              it = (int)(L / ((unsigned)nkt * (unsigned)njt));
    const int k0 = kt * CKW, j0 = jt * PTJ, i0 = it * A.chunk;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    const int row = wv - 1;
    const bool upd = row >= 0 && row < PTJ;
    const int jg = (j0 + row) & m;
    const size_t plane = (size_t)1 << (2 * lg);
    const size_t rowbase = (size_t)jg << lg;
    const size_t kk = (size_t)(k0 + 2 * lane), kh2 = (size_t)(k0 / 2 + lane);
    auto pb = [&](int pl) { return (size_t)(pl & m) * plane + rowbase; };
    auto ld_split = [&](const float *a, int pl) {  // both cells of the pair from the two colour halves
        const size_t q = pb(pl) + kh2;
        const bool odd = ((pl + jg) & 1) != 0;
        return make_float2(a[q + (odd ? hN : 0)], a[q + (odd ? 0 : hN)]);
    };
    // k-halo: lanes 0..2 PTJ - 1 of wave 0 serve row lane / 2, end lane & 1 (0: k0 - 1, 1: k0 + CKW)
    const bool kh = wv == 0 && lane < 2 * PTJ;
    const int khq = (lane & (2 * PTJ - 1)) >> 1, khs = lane & 1;
    const int khj = (j0 + khq) & m, khk = khs ? ((k0 + CKW) & m) : ((k0 - 1) & m);
    auto kh_u = [&](int pl) { return (size_t)(pl & m) * plane + ((size_t)khj << lg) + (size_t)khk; };
    auto kh_e = [&](int pl) {
        return (size_t)(pl & m) * plane + ((size_t)khj << lg) + ((size_t)(((pl & m) + khj + khk) & 1) << (lg - 1)) +
               (size_t)(khk >> 1);
    };
    auto slot = [&](int r, int l, int col) { return ((r + 1) * CLW + l + 1) * 2 + col; };

    Cell4 p0, p1, c0, c1;
    {
        const float2 um = *reinterpret_cast<const float2 *>(A.u + pb(i0 - 1) + kk), em = ld_split(A.e, i0 - 1);
        const float2 u0 = *reinterpret_cast<const float2 *>(A.u + pb(i0) + kk), e0 = ld_split(A.e, i0);
        p0 = mx_cell(um.x, em.x);
        p1 = mx_cell(um.y, em.y);
        c0 = mx_cell(u0.x, e0.x);
        c1 = mx_cell(u0.y, e0.y);
    }
    // raw loads of step p: u, e of plane p + 1; r and the k-halo cell of plane p
    struct Raw {
        float2 u, e, r;
        float khu, khe;
    };
    auto load = [&](int p) {
        Raw w;
        w.u = *reinterpret_cast<const float2 *>(A.u + pb(p + 1) + kk);
        w.e = ld_split(A.e, p + 1);
        w.r = ld_split(A.r, p);  // halo rows: loaded, not used
        w.khu = A.u[kh_u(p)];
        w.khe = A.e[kh_e(p)];
        return w;
    };
    Raw ra = load(i0), rb;  // issued one step ahead (more would cost occupancy here)
    int buf = 0;
    float se = 0.f, su = 0.f, sr = 0.f;
    auto step = [&](int p, bool second, const Raw &cur, Raw &nxt) {
        nxt = load(p + 1);
        const Cell4 n0 = mx_cell(cur.u.x, cur.e.x), n1 = mx_cell(cur.u.y, cur.e.y);
        float4 *B = sB + buf * (PTJ + 2) * CLW * 2;
        B[slot(row, lane, 0)] = pack(c0);
        B[slot(row, lane, 1)] = pack(c1);
        if (kh) B[khs ? slot(khq, CKW / 2, 0) : slot(khq, -1, 1)] = pack(mx_cell(cur.khu, cur.khe));
        __syncthreads();
        if (upd) {
            const Cell4 up0 = unpack(B[slot(row - 1, lane, 0)]), up1 = unpack(B[slot(row - 1, lane, 1)]);
            const Cell4 dn0 = unpack(B[slot(row + 1, lane, 0)]), dn1 = unpack(B[slot(row + 1, lane, 1)]);
            const Cell4 lf = unpack(B[slot(row, lane - 1, 1)]), rt = unpack(B[slot(row, lane + 1, 0)]);
            const float N0 = mx_nval(c0, p0, n0, up0, dn0, lf, c1, A.kc);
            const float N1 = mx_nval(c1, p1, n1, up1, dn1, c0, rt, A.kc);
            se += c0.e + c1.e;
            su += c0.u + c1.u;
            sr += (cur.r.x - N0) + (cur.r.y - N1);
        }
        if (second) {
            if (upd && (row & 1)) sR[row >> 1][lane] = make_float4(se, su, sr, 0.f);
            __syncthreads();
            if (upd && !(row & 1)) {
                const float4 o = sR[row >> 1][lane];
                const int I = (p & m) >> 1, J = jg >> 1, K = k0 / 2 + lane;
                const size_t nat = ((((size_t)I << lgc) + (size_t)J) << lgc) + (size_t)K;
                const size_t spl = A.split_c ? ((((size_t)I << lgc) + (size_t)J) << lgc) +
                                                   ((size_t)((I + J + K) & 1) << (lgc - 1)) + (size_t)(K >> 1)
                                             : nat;
                A.ebc[spl] = 0.125f * (se + o.x);
                A.uc[nat] = 0.125f * (su + o.y);
                A.rc[spl] = 0.125f * (sr + o.z);
            }
            se = su = sr = 0.f;
        }
        p0 = c0;
        p1 = c1;
        c0 = n0;
        c1 = n1;
        buf ^= 1;
    };
    for (int p = i0; p < i0 + A.chunk; p += 2) {
        step(p, false, ra, rb);
        step(p + 1, true, rb, ra);
    }
}

// ------------------------------------------------------------------- kernels

__global__ __launch_bounds__(kBlock) void k_mx_sweep_half(float *__restrict__ e, const float *__restrict__ u,
                                                            const float *__restrict__ r, int lg, int colour,
                                                            MxConst kc)
{
    mx_sweep_cell(e, u, r, (size_t)blockIdx.x * kBlock + threadIdx.x, lg, colour, kc);
}

// H half-sweeps of the 32^3 or 64^3 level in one launch, out of place: the
// geometry of the float64 k_sweep_tile, cells in LDS as {e, X, u, w}.  Each update
// is that of k_mx_sweep_half, bit by bit.
// Bound: the launch's latency and the updates, the surrounding rows included.
// 32^3, two sweeps: four launches of 3.4 us (and the gaps) -> 5.9 us; 64^3, one
// sweep: two of 3.5 us -> 4.7 us (two sweeps per launch: 10.3 us).
template <int LG, int H, bool PRO>
__global__ __launch_bounds__(1024) void k_mx_sweep_tile(const float *__restrict__ e, const float *__restrict__ u,
                                                        const float *__restrict__ r, float *__restrict__ out, MxConst kc,
                                                        const float *__restrict__ ec, const float *__restrict__ eb,
                                                        int mode)
{
    using P = TileProlong<float, LG, 4 + 2 * H>;
    __shared__ float sd[PRO ? P::CELLS : 1];
    constexpr int N = 1 << LG, M = N - 1, E = 4 + 2 * H, HALF = N / 2, NT = 1024;
    __shared__ float4 sc[E * E * N];
    const int t = threadIdx.x;
    const int i0 = 4 * (int)(blockIdx.x / (N / 4)) - H, j0 = 4 * (int)(blockIdx.x % (N / 4)) - H;
    auto slot = [](int i, int j, int k) { return ((i * E + j) << LG) + (k & 1) * HALF + (k >> 1); };
    auto cell = [&](int i, int j, int k) { return ix((i0 + i) & M, (j0 + j) & M, k, LG); };
    // the cell of thread t, round q, of half-sweep h: (4 + 2 m)^2 rows of N / 2 cells, m = H - 1 - h
    auto place = [&](int h, int q, int &i, int &j, int &k) {
        const int m = H - 1 - h, D = 4 + 2 * m, c = t + q * NT, row = c / HALF;
        i = H - m + row / D;
        j = H - m + row % D;
        k = 2 * (c % HALF) + ((i0 + i + j0 + j + h) & 1);
        return row < D * D;
    };
    constexpr int R = ((4 + 2 * (H - 1)) * (4 + 2 * (H - 1)) * HALF + NT - 1) / NT;  // rounds of the first half-sweep
    float rv[H][R];
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
        for (int q = 0; q < R; ++q) {
            int i, j, k;
            rv[h][q] = place(h, q, i, j, k) ? r[cell(i, j, k)] : 0.f;
        }
    constexpr int RL = (E * E * N + NT - 1) / NT;
    float xe[RL], xu[RL];
#pragma unroll
    for (int q = 0; q < RL; ++q) {
        const int c = t + q * NT, row = c >> LG;
        const size_t g = cell(row / E, row % E, c & M);  // in the mesh for any row
        xe[q] = e[g];
        xu[q] = u[g];
    }
    if constexpr (PRO) {
        P::template load<NT>(sd, ec, eb, i0, j0);
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < RL; ++q) {
        const int c = t + q * NT, row = c >> LG, k = c & M;
        if (row < E * E) {
            if (PRO) xe[q] += P::value(sd, row / E, row % E, k, mode);
            sc[slot(row / E, row % E, k)] = make_float4(xe[q], fexpm1(xe[q]), xu[q], fexp(xu[q]));
        }
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < H; ++h) {
#pragma unroll
        for (int q = 0; q < R; ++q) {
            int i, j, k;
            if (place(h, q, i, j, k)) {
                const int c = slot(i, j, k), side = ((i * E + j) << LG) + (1 - (k & 1)) * HALF;
                const float4 x = sc[c];
                const float4 n[6] = {sc[c + E * N], sc[c - E * N], sc[c + N], sc[c - N],
                                     sc[side + (((k + 1) & M) >> 1)], sc[side + (((k - 1) & M) >> 1)]};
                float en[6], Xn[6], un[6], wn[6];
#pragma unroll
                for (int s = 0; s < 6; ++s) {
                    en[s] = n[s].x;
                    Xn[s] = n[s].y;
                    un[s] = n[s].z;
                    wn[s] = n[s].w;
                }
                const float ne = x.x + mx_step(x.x, x.y, x.z, x.w, en, Xn, un, wn, rv[h][q], kc);
                sc[c] = make_float4(ne, fexpm1(ne), x.z, x.w);
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < (16 * N + NT - 1) / NT; ++q) {
        const int c = t + q * NT, row = c >> LG, k = c & M;
        if (row < 16) out[cell(H + (row >> 2), H + (row & 3), k)] = sc[slot(H + (row >> 2), H + (row & 3), k)].x;
    }
}

__global__ __launch_bounds__(kBlock) void k_mx_residual_restrict(const float *__restrict__ e,
                                                                   const float *__restrict__ u,
                                                                   const float *__restrict__ r, int lg, MxConst kc,
                                                                   float *__restrict__ eb_c, float *__restrict__ u_c,
                                                                   float *__restrict__ r_c, bool split, bool split_c)
{
    const int lgc = lg - 1;
    const size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x;
    const int K = (int)(t & ((1u << lgc) - 1)), J = (int)((t >> lgc) & ((1u << lgc) - 1)), I = (int)(t >> (2 * lgc));
    float em, um, rm;
    mx_restrict_block(e, u, r, I, J, K, lg, kc, em, um, rm, split);
    const size_t tc = sx(I, J, K, lgc, split_c);
    eb_c[tc] = em;
    u_c[t] = um;
    r_c[tc] = rm;
}

// r_c += N_c(eb); e_c = eb
__global__ __launch_bounds__(kBlock) void k_mx_coarse_rhs(const float *__restrict__ eb, const float *__restrict__ u,
                                                            int lg, MxConst kc, float *__restrict__ rc,
                                                            float *__restrict__ ec, bool split)
{
    const size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x;
    const int m = (1 << lg) - 1;
    const int k = (int)(t & m), j = (int)((t >> lg) & m), i = (int)(t >> (2 * lg));
    const size_t ts = sx(i, j, k, lg, split);
    rc[ts] += mx_value_at(eb, u, i, j, k, lg, kc, split);
    ec[ts] = eb[ts];
}

// one thread per coarse cell: its 8 daughters of the 2^lg mesh
__global__ __launch_bounds__(kBlock) void k_mx_prolong_add(float *__restrict__ e, const float *__restrict__ ec,
                                                             const float *__restrict__ eb, int lg, int mode, bool split,
                                                             bool split_c)
{
    const int lgc = lg - 1, m = (1 << lgc) - 1;
    const size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x;
    const int K = (int)(t & ((1u << lgc) - 1)), J = (int)((t >> lgc) & ((1u << lgc) - 1)), I = (int)(t >> (2 * lgc));
    auto d = [&](int i, int j, int k) {
        const size_t q = sx(i, j, k, lgc, split_c);
        return ec[q] - eb[q];
    };
    const float v0 = d(I, J, K);
    float gx = 0.f, gy = 0.f, gz = 0.f;
    if (mode == 0) {
        gx = d((I + 1) & m, J, K) - d((I - 1) & m, J, K);
        gy = d(I, (J + 1) & m, K) - d(I, (J - 1) & m, K);
        gz = d(I, J, (K + 1) & m) - d(I, J, (K - 1) & m);
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                float v = v0;
                if (mode == 0) {
                    v += (a ? 0.125f : -0.125f) * gx;
                    v += (b ? 0.125f : -0.125f) * gy;
                    v += (c ? 0.125f : -0.125f) * gz;
                }
                e[sx(2 * I + a, 2 * J + b, 2 * K + c, lg, split)] += v;
            }
}

// The tail (16^3, 8^3, 4^3) in one workgroup, every level in LDS as
// (e, expm1 e, u, e^u) per cell, so that an update reads its neighbours'
// exponentials and evaluates one of its own.  Layout and threads: TailGrid;
// the arithmetic is that of the other float32 levels (mx_step, mx_value).
// Bound: the latency of some 100 dependent half-sweeps.  V(4,4) cycle: 103 us
// with e, u and r alone in LDS (14 exponentials per update), now 58 us.
struct MxTail {
    float *e;             // top level, in and out
    const float *u, *r;
    float ih2[3];         // 16^3, 8^3, 4^3
    int lg0, pre, post, coarse, mode;
    float bC, q, max_du, omega;
};

template <int LG>
struct MxTailLevel : TailGrid<LG> {
    float4 *c;      // (e, expm1 e, u, e^u)
    float *r, *eb;
};

__device__ __forceinline__ float mx_tail_step(const float4 &c, const float4 n[6], float r, const MxConst &kc)
{
    const float en[6] = {n[0].x, n[1].x, n[2].x, n[3].x, n[4].x, n[5].x};
    const float Xn[6] = {n[0].y, n[1].y, n[2].y, n[3].y, n[4].y, n[5].y};
    const float un[6] = {n[0].z, n[1].z, n[2].z, n[3].z, n[4].z, n[5].z};
    const float wn[6] = {n[0].w, n[1].w, n[2].w, n[3].w, n[4].w, n[5].w};
    return c.x + mx_step(c.x, c.y, c.z, c.w, en, Xn, un, wn, r, kc);
}

// N(e) at a cell of a tail level
template <int LG>
__device__ __forceinline__ float mx_tail_value(const MxTailLevel<LG> &T, int i, int j, int k, const float4 &c,
                                               const MxConst &kc)
{
    using G = TailGrid<LG>;
    constexpr int M = G::M;
    const float4 n[6] = {T.c[G::slot((i + 1) & M, j, k)], T.c[G::slot((i - 1) & M, j, k)],
                         T.c[G::slot(i, (j + 1) & M, k)], T.c[G::slot(i, (j - 1) & M, k)],
                         T.c[G::slot(i, j, (k + 1) & M)], T.c[G::slot(i, j, (k - 1) & M)]};
    const float en[6] = {n[0].x, n[1].x, n[2].x, n[3].x, n[4].x, n[5].x};
    const float Xn[6] = {n[0].y, n[1].y, n[2].y, n[3].y, n[4].y, n[5].y};
    const float un[6] = {n[0].z, n[1].z, n[2].z, n[3].z, n[4].z, n[5].z};
    const float wn[6] = {n[0].w, n[1].w, n[2].w, n[3].w, n[4].w, n[5].w};
    return mx_value(c.x, c.y, c.z, c.w, en, Xn, un, wn, kc);
}

// Red-black sweeps of the 16^3 or 8^3 level.
template <int LG>
__device__ __forceinline__ void mx_tail_sweeps(const MxTailLevel<LG> &T, int sweeps, const MxConst &kc)
{
    using G = TailGrid<LG>;
    constexpr int W = G::W, M = G::M;
    const bool own = threadIdx.x < G::THREADS;
    int i = 0, j = 0, k0 = 0;
    float4 x[W];
    float r[W];
    if (own) {
        G::cell(threadIdx.x, i, j, k0);
#pragma unroll
        for (int c = 0; c < W; ++c) {
            x[c] = T.c[G::slot(i, j, k0 + c)];
            r[c] = T.r[G::slot(i, j, k0 + c)];
        }
    }
    const int par = __builtin_amdgcn_readfirstlane((i + j) & 1);  // uniform over the wave
    const int ip = (i + 1) & M, im = (i - 1) & M, jp = (j + 1) & M, jm = (j - 1) & M;
    // update columns B, B + 2, ... of the thread's cells
    auto half = [&](auto Bc) {
        constexpr int B = decltype(Bc)::value;
        const float4 out = T.c[G::slot(i, j, B ? (k0 + W) & M : (k0 - 1) & M)];
#pragma unroll
        for (int c = B; c < W; c += 2) {
            const int k = k0 + c;
            const float4 n[6] = {T.c[G::slot(ip, j, k)], T.c[G::slot(im, j, k)], T.c[G::slot(i, jp, k)],
                                 T.c[G::slot(i, jm, k)], c == W - 1 ? out : x[(c + 1) % W], c == 0 ? out : x[(c + W - 1) % W]};
            x[c].x = mx_tail_step(x[c], n, r[c], kc);
            x[c].y = fexpm1(x[c].x);
        }
#pragma unroll
        for (int c = B; c < W; c += 2) T.c[G::slot(i, j, k0 + c)] = x[c];
    };
    for (int h = 0; h < 2 * sweeps; ++h) {
        if (own) {
            if ((par ^ h) & 1)
                half(std::integral_constant<int, 1>{});
            else
                half(std::integral_constant<int, 0>{});
        }
        __syncthreads();
    }
}

// Sweeps of the 4^3 level by the first wave: within one wave the LDS accesses
// of a half-sweep are done before the next one's (wave_lds_sync).
__device__ __forceinline__ void mx_tail_sweeps4(const MxTailLevel<2> &T, int sweeps, const MxConst &kc)
{
    using G = TailGrid<2>;
    if (threadIdx.x < 64) {
        int i, j, k;
        G::cell(threadIdx.x, i, j, k);
        const int c = G::slot(i, j, k), par = (i + j + k) & 1;
        const int s[6] = {G::slot((i + 1) & 3, j, k), G::slot((i - 1) & 3, j, k), G::slot(i, (j + 1) & 3, k),
                          G::slot(i, (j - 1) & 3, k), G::slot(i, j, (k + 1) & 3), G::slot(i, j, (k - 1) & 3)};
        float4 x = T.c[c];
        const float r = T.r[c];
        for (int h = 0; h < 2 * sweeps; ++h) {
            if (par == (h & 1)) {
                const float4 n[6] = {T.c[s[0]], T.c[s[1]], T.c[s[2]], T.c[s[3]], T.c[s[4]], T.c[s[5]]};
                x.x = mx_tail_step(x, n, r, kc);
                x.y = fexpm1(x.x);
                T.c[c] = x;
            }
            wave_lds_sync();
        }
    }
    __syncthreads();
}

// Means of e, u and r - N(e) over the eight daughters, then the coarse source
// r_c += N_c(eb) and e_c = eb.
template <int LG>
__device__ __forceinline__ void mx_tail_restrict(const MxTailLevel<LG> &T, const MxTailLevel<LG - 1> &C,
                                                 const MxConst &kf, const MxConst &kcc)
{
    using G = TailGrid<LG>;
    using GC = TailGrid<LG - 1>;
    const int t = threadIdx.x;
    const int I = t >> (2 * LG - 2), J = (t >> (LG - 1)) & GC::M, K = t & GC::M;
    float se = 0.f, su = 0.f, sr = 0.f;
    if (t < GC::CELLS) {
#pragma unroll
        for (int d = 0; d < 8; ++d) {
            const int i = 2 * I + (d >> 2), j = 2 * J + ((d >> 1) & 1), k = 2 * K + (d & 1), c = G::slot(i, j, k);
            const float4 x = T.c[c];
            se += x.x;
            su += x.z;
            sr += T.r[c] - mx_tail_value(T, i, j, k, x, kf);
        }
        const int c = GC::slot(I, J, K);
        const float em = 0.125f * se, um = 0.125f * su;
        C.eb[c] = em;
        C.c[c] = make_float4(em, fexpm1(em), um, fexp(um));
    }
    __syncthreads();
    if (t < GC::CELLS) {
        const int c = GC::slot(I, J, K);
        const float rm = 0.125f * sr;
        C.r[c] = rm + mx_tail_value(C, I, J, K, C.c[c], kcc);
    }
    __syncthreads();
}

// e += P(e_c - eb): the thread's cells from their W / 2 parents
template <int LG>
__device__ __forceinline__ void mx_tail_prolong(const MxTailLevel<LG> &T, const MxTailLevel<LG - 1> &C, int mode)
{
    using G = TailGrid<LG>;
    using GC = TailGrid<LG - 1>;
    constexpr int MC = GC::M;
    if (threadIdx.x < G::THREADS) {
        int i, j, k0;
        G::cell(threadIdx.x, i, j, k0);
        auto d = [&](int a, int b, int c) {
            const int s = GC::slot(a & MC, b & MC, c & MC);
            return C.c[s].x - C.eb[s];
        };
#pragma unroll
        for (int h = 0; h < G::W / 2; ++h) {
            const int I = i >> 1, J = j >> 1, K = (k0 >> 1) + h;
            float v0 = d(I, J, K), gz = 0.f;
            if (mode == 0) {
                v0 += ((i & 1) ? 0.125f : -0.125f) * (d(I + 1, J, K) - d(I - 1, J, K));
                v0 += ((j & 1) ? 0.125f : -0.125f) * (d(I, J + 1, K) - d(I, J - 1, K));
                gz = 0.125f * (d(I, J, K + 1) - d(I, J, K - 1));
            }
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int s = G::slot(i, j, k0 + 2 * h + c);
                float4 x = T.c[s];
                x.x += c ? v0 + gz : v0 - gz;
                x.y = fexpm1(x.x);
                T.c[s] = x;
            }
        }
    }
    __syncthreads();
}

__global__ __launch_bounds__(kTailThreads) void k_mx_tail(MxTail A)
{
    __shared__ float4 s_c[4096 + 512 + 64];
    __shared__ float s_r[4096 + 512 + 64], s_eb[512 + 64];
    const MxTailLevel<4> T4{{}, s_c, s_r, nullptr};
    const MxTailLevel<3> T3{{}, s_c + 4096, s_r + 4096, s_eb};
    const MxTailLevel<2> T2{{}, s_c + 4608, s_r + 4608, s_eb + 512};
    const MxConst k4{A.ih2[0], A.bC, A.q, A.max_du, A.omega}, k3{A.ih2[1], A.bC, A.q, A.max_du, A.omega},
        k2{A.ih2[2], A.bC, A.q, A.max_du, A.omega};
    const int lg = A.lg0, n0 = 1 << (3 * lg), m = (1 << lg) - 1;
    auto slot0 = [&](int c) {
        const int i = c >> (2 * lg), j = (c >> lg) & m, k = c & m;
        return lg == 4 ? TailGrid<4>::slot(i, j, k) : 4096 + TailGrid<3>::slot(i, j, k);
    };
    for (int c = threadIdx.x; c < n0; c += kTailThreads) {
        const float e = A.e[c], u = A.u[c];
        s_c[slot0(c)] = make_float4(e, fexpm1(e), u, fexp(u));
        s_r[slot0(c)] = A.r[c];
    }
    __syncthreads();
    if (lg == 4) {
        mx_tail_sweeps(T4, A.pre, k4);
        mx_tail_restrict(T4, T3, k4, k3);
    }
    mx_tail_sweeps(T3, A.pre, k3);
    mx_tail_restrict(T3, T2, k3, k2);
    mx_tail_sweeps4(T2, A.coarse, k2);
    mx_tail_prolong(T3, T2, A.mode);
    mx_tail_sweeps(T3, A.post, k3);
    if (lg == 4) {
        mx_tail_prolong(T4, T3, A.mode);
        mx_tail_sweeps(T4, A.post, k4);
    }
    for (int c = threadIdx.x; c < n0; c += kTailThreads) A.e[c] = s_c[slot0(c)].x;
}

// float64 residual of u on the finest level, its float32 copies for the inner
// cycle, and per-block max / sum of squares (thread per 2x2x2 block)
__global__ __launch_bounds__(kBlock) void k_mx_outer_residual(const double *__restrict__ u,
                                                                const double *__restrict__ f, int lg, OpConst kc,
                                                                float *__restrict__ r32, float *__restrict__ u32,
                                                                float *__restrict__ e32,
                                                                double *__restrict__ partial, int nparts, bool split)
{
    __shared__ double sh[2 * kBlock / 64];
    const int lgc = lg - 1;
    const size_t nblk = (size_t)1 << (3 * lgc);
    double mx = 0.0, sm = 0.0;
    for (size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x; t < nblk; t += (size_t)gridDim.x * kBlock) {
        const int K = (int)(t & ((1u << lgc) - 1)), J = (int)((t >> lgc) & ((1u << lgc) - 1)),
                  I = (int)(t >> (2 * lgc));
        BlockRes br;
        block_residuals(u, f, I, J, K, lg, kc, br);
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const size_t cc = ix(2 * I + a, 2 * J + b, 2 * K + c, lg);
                    const double r = br.r[(a * 2 + b) * 2 + c];
                    const size_t cs = sx(2 * I + a, 2 * J + b, 2 * K + c, lg, split);
                    r32[cs] = (float)r;
                    u32[cc] = (float)u[cc];
                    e32[cs] = 0.0f;
                    mx = nanmax_d(mx, fabs(r));
                    sm += r * r;
                }
    }
    for (int o = 32; o > 0; o >>= 1) {
        mx = nanmax_d(mx, __shfl_xor(mx, o, 64));
        sm += __shfl_xor(sm, o, 64);
    }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        sh[w] = mx;
        sh[kBlock / 64 + w] = sm;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < kBlock / 64; ++i) {
            mx = nanmax_d(mx, sh[i]);
            sm += sh[kBlock / 64 + i];
        }
        partial[blockIdx.x] = mx;
        partial[nparts + blockIdx.x] = sm;
    }
}

// Float64 outer step of the mixed solve on a level-0 mesh with N >= 64:
// v = u + e (ADD_E) or v = u, then r = f - L(v) at every cell.  Same plane
// march as the colour pass: workgroups of RTJ rows of a 64-cell row tile plus
// a halo row on each side (one wave per row, one cell per lane); v and e^v of
// a plane are staged in LDS, so every exponential is evaluated once per cell
// (plus the halo).  Writes v (ADD_E: into the second buffer uout), r and v as
// float32 for the inner cycle, and per-workgroup max|r| and sum r^2.  Every
// wave issues the same loads in every plane (see k_mx_colour).
constexpr int RTJ = 8, RTK = 64, RLW = RTK + 2;

struct CorrArgs {
    const double *u, *f;
    const float *e;
    double *uout;
    float *r32, *u32;
    int lg, chunk, nunits;
    bool split;
    OpConst kc;
    double *partial;
    int nparts;
    const double *exp2tab;
};

template <bool ADD_E>
__global__ __launch_bounds__(64 * (RTJ + 2)) void k_mx_correct_residual(CorrArgs A)
{
    __shared__ double2 sB[2 * (RTJ + 2) * RLW];
    __shared__ double red[2 * (RTJ + 2)];
    __shared__ double tab[64];
    if (threadIdx.x < 64) tab[threadIdx.x] = A.exp2tab[threadIdx.x];
    __syncthreads();
    const int lg = A.lg, m = (1 << lg) - 1;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    const int row = wv - 1;
    const bool upd = row >= 0 && row < RTJ;
    const size_t plane = (size_t)1 << (2 * lg);
    const int nkt = (1 << lg) / RTK, njt = (1 << lg) / RTJ;
    // k-halo duty: lanes 0..2 RTJ - 1 of wave 0 serve row lane / 2, side lane & 1
    const bool kh = wv == 0 && lane < 2 * RTJ;
    const int khq = (lane & (2 * RTJ - 1)) >> 1, khs = lane & 1;
    double mx = 0.0, sm = 0.0;
    for (int unit = blockIdx.x; unit < A.nunits; unit += gridDim.x) {
        const int kt = unit % nkt, jt = (unit / nkt) % njt, it = unit / (nkt * njt);
        const int k0 = kt * RTK, j0 = jt * RTJ, i0 = it * A.chunk;
        const int jg = (j0 + row) & m, k = k0 + lane;
        const size_t rowoff = ((size_t)jg << lg) + (size_t)k;
        const int khj = (j0 + khq) & m, khk = khs ? ((k0 + RTK) & m) : ((k0 - 1) & m);
        const size_t khoff = ((size_t)khj << lg) + (size_t)khk;
        auto eidx = [&](int pl, size_t off, int j, int kk) {
            return (size_t)(pl & m) * plane +
                   (A.split ? (((size_t)j << lg) + ((size_t)(((pl & m) + j + kk) & 1) << (lg - 1)) + (size_t)(kk >> 1))
                            : off);
        };
        auto vload = [&](int pl, size_t off, int j, int kk) {
            double v = A.u[(size_t)(pl & m) * plane + off];
            if (ADD_E) v += (double)A.e[eidx(pl, off, j, kk)];
            return v;
        };
        // raw loads of step p (u and e kept apart: they are summed where used,
        // so that no arithmetic on a load in flight sits at the loop latch)
        struct Raw {
            double u, f, ku;
            float e, ke;
        };
        auto load = [&](int p) {
            Raw w;
            w.u = A.u[(size_t)((p + 1) & m) * plane + rowoff];
            w.e = ADD_E ? A.e[eidx(p + 1, rowoff, jg, k)] : 0.f;
            w.f = A.f[(size_t)(p & m) * plane + rowoff];  // halo rows: loaded, not used
            w.ku = A.u[(size_t)(p & m) * plane + khoff];
            w.ke = ADD_E ? A.e[eidx(p, khoff, khj, khk)] : 0.f;
            return w;
        };
        double vm = vload(i0 - 1, rowoff, jg, k), vc = vload(i0, rowoff, jg, k);
        double Em = exp64(vm, tab), Ec = exp64(vc, tab);
        Raw ra = load(i0), rb = load(i0 + 1), rc, rd;  // issued two steps ahead (see k_mx_colour)
        int buf = 0;
        auto step = [&](int p, const Raw &cur, Raw &nxt) {
            nxt = load(p + 2);
            const double vp = cur.u + (double)cur.e, Ep = exp64(vp, tab);
            double2 *B = sB + buf * (RTJ + 2) * RLW;
            B[(row + 1) * RLW + lane + 1] = make_double2(vc, Ec);
            if (kh) {
                const double kv = cur.ku + (double)cur.ke;
                B[(khq + 1) * RLW + (khs ? RLW - 1 : 0)] = make_double2(kv, exp64(kv, tab));
            }
            __syncthreads();
            if (upd) {
                const double2 a = B[row * RLW + lane + 1], b = B[(row + 2) * RLW + lane + 1];
                const double2 c = B[(row + 1) * RLW + lane], d = B[(row + 1) * RLW + lane + 2];
                const double d0 = vp - vc, d1 = vm - vc, d2 = b.x - vc, d3 = a.x - vc, d4 = d.x - vc, d5 = c.x - vc;
                const double S1 = ((d0 + d1) + (d2 + d3)) + (d4 + d5);
                const double S3 = ((Ep * d0 + Em * d1) + (b.y * d2 + a.y * d3)) + (d.y * d4 + c.y * d5);
                const double L = A.kc.ih2 * 0.5 * (S3 + Ec * S1) + A.kc.bC * expm1_64(-A.kc.q * vc, tab);
                const double r = cur.f - L;
                const size_t o = (size_t)(p & m) * plane + rowoff;
                if (ADD_E) A.uout[o] = vc;
                A.u32[o] = (float)vc;
                A.r32[A.split ? (size_t)(p & m) * plane + ((size_t)jg << lg) + ((size_t)(((p & m) + jg + k) & 1) << (lg - 1)) + (size_t)(k >> 1) : o] = (float)r;
                mx = nanmax_d(mx, fabs(r));
                sm += r * r;
            }
            vm = vc;
            Em = Ec;
            vc = vp;
            Ec = Ep;
            buf ^= 1;
        };
        for (int p = i0; p < i0 + A.chunk; p += 4) {
            step(p, ra, rc);
            step(p + 1, rb, rd);
            step(p + 2, rc, ra);
            step(p + 3, rd, rb);
        }
        __syncthreads();  // the next unit reuses the LDS buffers
    }
    for (int o = 32; o > 0; o >>= 1) {
        mx = nanmax_d(mx, __shfl_xor(mx, o, 64));
        sm += __shfl_xor(sm, o, 64);
    }
    if (lane == 0) {
        red[wv] = mx;
        red[RTJ + 2 + wv] = sm;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < RTJ + 2; ++w) {
            mx = nanmax_d(mx, red[w]);
            sm += red[RTJ + 2 + w];
        }
        A.partial[blockIdx.x] = mx;
        A.partial[A.nparts + blockIdx.x] = sm;
    }
}

__global__ __launch_bounds__(kBlock) void k_mx_update(double *__restrict__ u, const float *__restrict__ e, int lg,
                                                        bool split)
{
    const size_t n = (size_t)1 << (3 * lg);
    const int m = (1 << lg) - 1;
    for (size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x; t < n; t += (size_t)gridDim.x * kBlock) {
        const int k = (int)(t & m), j = (int)((t >> lg) & m), i = (int)(t >> (2 * lg));
        u[t] += (double)e[sx(i, j, k, lg, split)];
    }
}

__global__ __launch_bounds__(1024) void k_mx_final(const double *__restrict__ partial, int nparts,
                                                    double *__restrict__ out)
{
    __shared__ double sh[32];
    double mx = 0.0, sm = 0.0;
    for (int i = threadIdx.x; i < nparts; i += 1024) {
        mx = nanmax_d(mx, partial[i]);
        sm += partial[nparts + i];
    }
    for (int o = 32; o > 0; o >>= 1) {
        mx = nanmax_d(mx, __shfl_xor(mx, o, 64));
        sm += __shfl_xor(sm, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        sh[threadIdx.x >> 6] = mx;
        sh[16 + (threadIdx.x >> 6)] = sm;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < 16; ++i) {
            mx = nanmax_d(mx, sh[i]);
            sm += sh[16 + i];
        }
        out[0] = mx;
        out[1] = sm;
    }
}

inline unsigned nb(size_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

MxConst mx_const(const mgfr_ctx *c, int l)
{
    return MxConst{(float)(1.0 / (c->lev[l].h * c->lev[l].h)), (float)c->bC, (float)c->q, (float)c->p.max_du,
                   (float)c->omega_now};
}

// Levels swept by the one-colour pass kernel store e, r and ebar split by colour.
static bool split_level(const mgfr_ctx *c, int l) { return c->colour32_min_n > 0 && c->lev[l].N >= c->colour32_min_n; }

// Per-launch timing of the finest level's sweep kernels: a pair of events
// around each launch (read back by collect_timing).
static int timer_slot(mgfr_ctx *c, bool timed, int &slot)
{
    slot = -1;
    if (!timed) return MGFR_OK;
    Timer &T = c->sweep_timer;
    if (T.used + 2 > (int)T.ev.size())
        for (int q = 0; q < 16; ++q) {
            hipEvent_t ev;
            MGFR_HIP(hipEventCreate(&ev));
            T.ev.push_back(ev);
        }
    slot = T.used;
    T.used += 2;
    MGFR_HIP(hipEventRecord(T.ev[slot], c->stream));
    return MGFR_OK;
}

static int timer_end(mgfr_ctx *c, int slot)
{
    if (slot >= 0) MGFR_HIP(hipEventRecord(c->sweep_timer.ev[slot + 1], c->stream));
    return MGFR_OK;
}

// 32^3 and 64^3, unless they run one kernel per colour: see k_mx_sweep_tile
static bool tile_level(const mgfr_ctx *c, const Level &L)
{
    return c->fused32 && (L.N == 32 || L.N == 64) && L.e32alt != nullptr;
}

// With `from` (tile levels, at least one sweep) the correction of that coarser
// level is added first.
int mx_launch_sweeps(mgfr_ctx *c, int l, int sweeps, bool timed, const Level *from = nullptr)
{
    Level &L = c->lev[l];
    const MxConst kc = mx_const(c, l);
    const size_t half = (size_t)1 << (3 * L.lg - 1);
    const bool colour_pass = split_level(c, l);
    const bool tile = tile_level(c, L);  // one sweep of 64^3 or two of 32^3 per launch
    int slot, rc;
    for (int s = 0; s < sweeps; ++s) {
        if (colour_pass && c->fused32 && L.N >= kFusedMin32) {
            const unsigned nkt = (unsigned)(L.N / kRowW), njt = (unsigned)((L.N + kRowI - 1) / kRowI);
            const int chunk = row_chunk(L.N, nkt * njt);
            const SweepRowsArgs A{L.e32, L.e32alt, L.u32, L.r32, L.lg, chunk, nkt, njt, kc};
            const unsigned nbf = nkt * njt * (unsigned)((L.N + chunk - 1) / chunk);
            if (l == 0 && c->e32_zero) {  // first sweep after a float64 check; not timed
                k_mx_sweep_rows<true><<<nbf, 64 * (kRowF + 1), 0, c->stream>>>(A);
                c->e32_zero = false;
            } else {
                if ((rc = timer_slot(c, timed, slot))) return rc;
                k_mx_sweep_rows<false><<<nbf, 64 * (kRowF + 1), 0, c->stream>>>(A);
                if ((rc = timer_end(c, slot))) return rc;
            }
            std::swap(L.e32, L.e32alt);
        } else if (colour_pass) {
            const int chunk = colour_chunk(L.N);
            const unsigned nb = (unsigned)((L.N / CKW) * ((L.N + CTJ - 1) / CTJ) * (L.N / chunk));
            for (int colour = 0; colour < 2; ++colour) {
                const ColourArgs A{L.e32, L.u32, L.r32, L.lg, colour, chunk, kc};
                if (l == 0 && c->e32_zero) {  // first pass after a float64 check; not timed
                    k_mx_colour_zero<<<nb, 64 * (CTJ + 2), 0, c->stream>>>(A);
                    c->e32_zero = false;
                    continue;
                }
                if ((rc = timer_slot(c, timed, slot))) return rc;
                k_mx_colour<<<nb, 64 * (CTJ + 2), 0, c->stream>>>(A);
                if ((rc = timer_end(c, slot))) return rc;
            }
        } else if (tile) {
            const unsigned nbt = (unsigned)((L.N / 4) * (L.N / 4));
            const bool two = L.N == 32 && !timed && s + 1 < sweeps;  // timing counts one sweep per launch
            if ((rc = timer_slot(c, timed, slot))) return rc;
            auto go = [&](auto *plain, auto *prolong) {
                (from ? prolong : plain)<<<nbt, 1024, 0, c->stream>>>(L.e32, L.u32, L.r32, L.e32alt, kc,
                                                                      from ? from->e32 : nullptr,
                                                                      from ? from->ebar32 : nullptr, c->p.prolong);
            };
            if (L.N == 64)
                go(k_mx_sweep_tile<6, 2, false>, k_mx_sweep_tile<6, 2, true>);
            else if (two)
                go(k_mx_sweep_tile<5, 4, false>, k_mx_sweep_tile<5, 4, true>);
            else
                go(k_mx_sweep_tile<5, 2, false>, k_mx_sweep_tile<5, 2, true>);
            from = nullptr;
            if ((rc = timer_end(c, slot))) return rc;
            std::swap(L.e32, L.e32alt);
            if (two) ++s;
        } else {
            for (int colour = 0; colour < 2; ++colour) {
                if ((rc = timer_slot(c, timed, slot))) return rc;
                k_mx_sweep_half<<<nb(half), kBlock, 0, c->stream>>>(L.e32, L.u32, L.r32, L.lg, colour, kc);
                if ((rc = timer_end(c, slot))) return rc;
            }
        }
    }
    MGFR_HIP(hipGetLastError());
    return MGFR_OK;
}

int mx_launch_tail(mgfr_ctx *c, int l0)
{
    const Level &L = c->lev[l0];
    MxTail A;
    A.e = L.e32;
    A.u = L.u32;
    A.r = L.r32;
    A.lg0 = L.lg;  // 4 or 3: meshes have at least 8 cells a side
    for (int k = 0; k < 3; ++k) {
        const double h = c->p.box / (16 >> k);
        A.ih2[k] = (float)(1.0 / (h * h));
    }
    A.pre = c->p.pre_smooth;
    A.post = c->p.post_smooth;
    A.coarse = c->p.coarse_sweeps;
    A.mode = c->p.prolong;
    A.bC = (float)c->bC;
    A.q = (float)c->q;
    A.max_du = (float)c->p.max_du;
    A.omega = (float)c->omega_now;
    k_mx_tail<<<1, kTailThreads, 0, c->stream>>>(A);
    MGFR_HIP(hipGetLastError());
    return MGFR_OK;
}

int mx_vcycle(mgfr_ctx *c, int l)
{
    Level &L = c->lev[l];
    if (L.N <= kTailN) return mx_launch_tail(c, l);
    int rc;
    if ((rc = mx_launch_sweeps(c, l, c->p.pre_smooth, l == 0 && c->timing))) return rc;
    Level &Lc = c->lev[l + 1];
    const size_t nc = (size_t)1 << (3 * Lc.lg);
    const bool sf = split_level(c, l), sc = split_level(c, l + 1);
    if (sf && L.N >= CKW) {
        const int chunk = L.N / 8;
        const unsigned nbk = (unsigned)((L.N / CKW) * (L.N / PTJ) * (L.N / chunk));
        k_mx_restrict_pass<<<nbk, 64 * (PTJ + 2), 0, c->stream>>>(
            RestrictArgs{L.e32, L.u32, L.r32, Lc.ebar32, Lc.u32, Lc.r32, L.lg, chunk, sc, mx_const(c, l)});
    } else {
        k_mx_residual_restrict<<<nb(nc), kBlock, 0, c->stream>>>(L.e32, L.u32, L.r32, L.lg, mx_const(c, l),
                                                                 Lc.ebar32, Lc.u32, Lc.r32, sf, sc);
    }
    k_mx_coarse_rhs<<<nb(nc), kBlock, 0, c->stream>>>(Lc.ebar32, Lc.u32, Lc.lg, mx_const(c, l + 1), Lc.r32, Lc.e32,
                                                      sc);
    MGFR_HIP(hipGetLastError());
    if ((rc = mx_vcycle(c, l + 1))) return rc;
    const bool with_sweep = tile_level(c, L) && c->p.post_smooth > 0;
    if (!with_sweep) {
        k_mx_prolong_add<<<nb(nc), kBlock, 0, c->stream>>>(L.e32, Lc.e32, Lc.ebar32, L.lg, c->p.prolong, sf, sc);
        MGFR_HIP(hipGetLastError());
    }
    return mx_launch_sweeps(c, l, c->p.post_smooth, l == 0 && c->timing, with_sweep ? &Lc : nullptr);
}

}  // namespace

int mixed_alloc(mgfr_ctx *c)
{
    for (int l = 0; l < c->nlev; ++l) {
        Level &L = c->lev[l];
        const size_t bytes = sizeof(float) * (size_t)L.N * L.N * L.N;
        MGFR_HIP(hipMalloc(&L.e32, bytes));
        MGFR_HIP(hipMalloc(&L.r32, bytes));
        MGFR_HIP(hipMalloc(&L.u32, bytes));
        if (l > 0) MGFR_HIP(hipMalloc(&L.ebar32, bytes));
        if (L.N >= 32) MGFR_HIP(hipMalloc(&L.e32alt, bytes));
    }
    return MGFR_OK;
}

// Float64 residual of the level-0 iterate (also prepares the float32 inner
// problem); returns max|r| and sum r^2 on the host.
static int outer_residual(mgfr_ctx *c, double *rmax, double *rsq)
{
    Level &L0 = c->lev[0];
    const size_t nblk = (size_t)1 << (3 * (L0.lg - 1));
    const unsigned g = (unsigned)std::min<size_t>(nb(nblk), (size_t)c->nparts);
    k_mx_outer_residual<<<g, kBlock, 0, c->stream>>>(L0.u, L0.f, L0.lg, level_const(c, 0), L0.r32, L0.u32, L0.e32,
                                                      c->partial, (int)g, split_level(c, 0));
    k_mx_final<<<1, 1024, 0, c->stream>>>(c->partial, (int)g, c->dscal);
    MGFR_HIP(hipGetLastError());
    MGFR_HIP(hipMemcpyAsync(c->hscal, c->dscal, 2 * sizeof(double), hipMemcpyDeviceToHost, c->stream));
    MGFR_HIP(hipStreamSynchronize(c->stream));
    *rmax = c->hscal[0];
    *rsq = c->hscal[1];
    return MGFR_OK;
}

// Outer step: (add_e) u <- u + e, then the float64 residual of u, the inner
// problem's float32 arrays and e = 0; returns max|r| and sum r^2 on the host.
// On meshes with N >= 64 one plane-marching kernel does both (the new iterate
// goes to the second level-0 buffer, which then becomes the current one).
static int outer_step(mgfr_ctx *c, bool add_e, double *rmax, double *rsq)
{
    Level &L0 = c->lev[0];
    const size_t n = (size_t)L0.N * L0.N * L0.N;
    if (L0.N < RTK || L0.alt == nullptr) {
        if (add_e)
            k_mx_update<<<(unsigned)std::min<size_t>(nb(n), 8192), kBlock, 0, c->stream>>>(L0.u, L0.e32, L0.lg,
                                                                                            split_level(c, 0));
        MGFR_HIP(hipGetLastError());
        return outer_residual(c, rmax, rsq);
    }
    CorrArgs A;
    A.u = L0.u;
    A.f = L0.f;
    A.e = L0.e32;
    A.uout = add_e ? L0.alt : nullptr;
    A.r32 = L0.r32;
    A.u32 = L0.u32;
    A.lg = L0.lg;
    A.chunk = L0.N / 8;
    A.nunits = (L0.N / RTK) * (L0.N / RTJ) * 8;
    A.split = split_level(c, 0);
    A.kc = level_const(c, 0);
    A.partial = c->partial;
    A.exp2tab = c->exp2tab;
    const int g = std::min(A.nunits, c->nparts);
    A.nparts = g;
    if (add_e)
        k_mx_correct_residual<true><<<g, 64 * (RTJ + 2), 0, c->stream>>>(A);
    else
        k_mx_correct_residual<false><<<g, 64 * (RTJ + 2), 0, c->stream>>>(A);
    if (add_e) std::swap(L0.u, L0.alt);
    // e = 0: cleared here, or by the first colour pass of the next cycle, which
    // then reads no e and writes the cells it does not update as 0
    c->e32_zero = split_level(c, 0) && c->p.pre_smooth >= 1;
    if (!c->e32_zero) MGFR_HIP(hipMemsetAsync(L0.e32, 0, n * sizeof(float), c->stream));
    k_mx_final<<<1, 1024, 0, c->stream>>>(c->partial, g, c->dscal);
    MGFR_HIP(hipGetLastError());
    MGFR_HIP(hipMemcpyAsync(c->hscal, c->dscal, 2 * sizeof(double), hipMemcpyDeviceToHost, c->stream));
    MGFR_HIP(hipStreamSynchronize(c->stream));
    *rmax = c->hscal[0];
    *rsq = c->hscal[1];
    return MGFR_OK;
}

int solve_mixed(mgfr_ctx *c, double *u, mgfr_stats *st, double D)
{
    Level &L0 = c->lev[0];
    const size_t n = (size_t)L0.N * L0.N * L0.N;
    const double ncell = (double)n;
    double rmax, rsq;
    int rc = outer_step(c, false, &rmax, &rsq);
    if (rc) return rc;
    double res = rmax / D, prev = res, prev2 = -1.0;  // prev, prev2: one and two checks back
    st->res0 = res;
    int it = 0, outer = 0, grow = 0, status;
    double rate = 0.5;  // residual reduction per correction cycle, from the last outer step
    c->omega_now = c->omega32;
    for (;;) {
        if (!std::isfinite(res) || grow >= 3) {
            // fall back: plain float64 solve from u = 0 (in the caller's array)
            L0.u = u;
            L0.alt = c->alt0;
            MGFR_HIP(hipMemsetAsync(u, 0, n * sizeof(double), c->stream));
            st->fell_back = 1;
            const int done = it;
            status = solve_fp64_from(c, st, D);
            st->outer_iters = done + st->vcycles;
            return status;
        }
        if (res <= c->p.tol) { status = MGFR_OK; break; }
        if (it >= c->p.max_vcycles) { status = MGFR_NOT_CONVERGED; break; }
        // Run up to inner_max correction cycles before the next float64
        // residual, but not past the cycle before the one the measured rate
        // predicts to reach the tolerance: each cycle is a full FAS V-cycle
        // of N_u(e) = r, so only the checks are skipped, and the last cycles
        // are checked one by one.
        int k = 1;
        if (c->inner_max > 1 && rate < 1.0) {
            const double need = std::ceil(std::log(c->p.tol / res) / std::log(rate));
            if (need > 2.0) k = (int)std::min<double>({(double)c->inner_max, need - 1.0, (double)(c->p.max_vcycles - it)});
        }
        for (int j = 0; j < k; ++j)
            if ((rc = mx_vcycle(c, 0))) return rc;
        if ((rc = outer_step(c, true, &rmax, &rsq))) return rc;
        if (c->timing && (rc = collect_timing(c, st))) return rc;
        prev2 = outer >= 1 ? prev : -1.0;
        prev = res;
        res = rmax / D;
        adapt_smoothing(c, res, prev2);
        if (res > 0.0 && prev > 0.0) rate = std::min(1.0, std::pow(res / prev, 1.0 / k));
        grow = (res > prev) ? grow + 1 : 0;
        if (grow) c->omega_now = 1.0;  // over-relaxation off for the rest of the solve once the residual grows
        if (outer < MGFR_MAX_HIST) st->res_hist[outer] = res;
        it += k;
        ++outer;
    }
    st->vcycles = it;
    st->outer_iters = outer;
    st->res = res;
    st->l2res = std::sqrt(rsq / ncell) / D;
    return status;
}

}  // namespace mgfr
