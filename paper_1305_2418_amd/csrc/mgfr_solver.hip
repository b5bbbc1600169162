// FP64 multigrid path of the f(R) field solve on gfx950.
//
// Operator (Sec. 3.2, Eq. u_discrete_field_eq, multiplied by a^2 to the
// comoving dimensionless form):
//   L_c(u) = (1/h^2) sum_nb (e^{u_nb} + e^{u_c})/2 (u_nb - u_c) - bC (1 - e^{-q u_c})
//   f_c    = beta Omega_m a^-3 delta_c,      q = 1/(n+1)
// Smoother: red-black Newton-Gauss-Seidel (Sec. 3.3, Eq. iterative_correction).
// Cycle: FAS V-cycle with 8-daughter-mean restriction, coarse source
// f_2h = L_2h(R u) + R(f - L_h u) and correction u += P(u_2h - R u)
// (Sec. 3.3, Eq. fine_correction), down to a 4^3 grid.
//
// Memory layout: every level is a dense N^3 float64 array in C order
// (k fastest).  Index arithmetic uses N = 2^lg.
#include "mgfr_internal.h"
#include "mgfr_ops.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <type_traits>

namespace mgfr {

// ------------------------------------------------------------------ errors

static thread_local std::string g_err;

int set_error(int code, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

int hip_fail(hipError_t e, const char *what, const char *file, int line)
{
    return set_error(e == hipErrorOutOfMemory ? MGFR_ERR_OOM : MGFR_ERR_HIP, "%s failed: %s (%s:%d)", what,
                     hipGetErrorString(e), file, line);
}

// ------------------------------------------------------------ device helpers

// Newton-Gauss-Seidel step for one cell from its value, its six neighbours and
// its source: -(L_c - f_c) / (dL_c/du_c), optionally limited to |du| <= max_du.
// With S1 = sum (u_n - u_c), S2 = sum e^{u_n}, S3 = sum e^{u_n} (u_n - u_c):
//   flux sum          = (S3 + e^{u_c} S1) / 2
//   d(flux sum)/du_c  = (e^{u_c} (S1 - 6) - S2) / 2
__device__ __forceinline__ double ngs_step(double uc, double n0, double n1, double n2, double n3,
                                           double n4, double n5, double f, const OpConst &k)
{
    double ec = exp64(uc, k.tab);
    double d0 = n0 - uc, d1 = n1 - uc, d2 = n2 - uc, d3 = n3 - uc, d4 = n4 - uc, d5 = n5 - uc;
    double e0 = exp64(n0, k.tab), e1 = exp64(n1, k.tab), e2 = exp64(n2, k.tab), e3 = exp64(n3, k.tab),
           e4 = exp64(n4, k.tab), e5 = exp64(n5, k.tab);
    double S1 = ((d0 + d1) + (d2 + d3)) + (d4 + d5);
    double S2 = ((e0 + e1) + (e2 + e3)) + (e4 + e5);
    double S3 = ((e0 * d0 + e1 * d1) + (e2 * d2 + e3 * d3)) + (e4 * d4 + e5 * d5);
    double em = expm1_64(-k.q * uc, k.tab);
    double L = k.ih2 * 0.5 * (S3 + ec * S1) + k.bC * em;
    double J = k.ih2 * 0.5 * (ec * (S1 - 6.0) - S2) - k.bC * k.q * (1.0 + em);
    double du = -(L - f) / J;
    if (k.max_du > 0.0) du = fmin(fmax(du, -k.max_du), k.max_du);
    return du;
}

__device__ __forceinline__ double op_value(double uc, double n0, double n1, double n2, double n3,
                                           double n4, double n5, const OpConst &k)
{
    double ec = exp64(uc, k.tab);
    double d0 = n0 - uc, d1 = n1 - uc, d2 = n2 - uc, d3 = n3 - uc, d4 = n4 - uc, d5 = n5 - uc;
    double e0 = exp64(n0, k.tab), e1 = exp64(n1, k.tab), e2 = exp64(n2, k.tab), e3 = exp64(n3, k.tab),
           e4 = exp64(n4, k.tab), e5 = exp64(n5, k.tab);
    double S1 = ((d0 + d1) + (d2 + d3)) + (d4 + d5);
    double S3 = ((e0 * d0 + e1 * d1) + (e2 * d2 + e3 * d3)) + (e4 * d4 + e5 * d5);
    return k.ih2 * 0.5 * (S3 + ec * S1) + k.bC * expm1_64(-k.q * uc, k.tab);
}

// L_c at (i,j,k) of a periodic 2^lg mesh.
__device__ __forceinline__ double op_at(const double *__restrict__ u, int i, int j, int k, int lg,
                                        const OpConst &kc)
{
    const int m = (1 << lg) - 1;
    double uc = u[cidx(i, j, k, lg)];
    return op_value(uc, u[cidx((i + 1) & m, j, k, lg)], u[cidx((i - 1) & m, j, k, lg)],
                    u[cidx(i, (j + 1) & m, k, lg)], u[cidx(i, (j - 1) & m, k, lg)],
                    u[cidx(i, j, (k + 1) & m, lg)], u[cidx(i, j, (k - 1) & m, lg)], kc);
}

// Update one cell of colour `colour` given its flat index t over that colour's cells.
__device__ __forceinline__ void sweep_cell(double *__restrict__ u, const double *__restrict__ f, size_t t,
                                           int lg, int colour, const OpConst &kc)
{
    const int m = (1 << lg) - 1;
    int mh = (int)(t & (size_t)((1 << (lg - 1)) - 1));
    size_t row = t >> (lg - 1);
    int j = (int)(row & m);
    int i = (int)(row >> lg);
    int k = 2 * mh + ((i + j + colour) & 1);
    size_t c = cidx(i, j, k, lg);
    double uc = u[c];
    double du = ngs_step(uc, u[cidx((i + 1) & m, j, k, lg)], u[cidx((i - 1) & m, j, k, lg)],
                         u[cidx(i, (j + 1) & m, k, lg)], u[cidx(i, (j - 1) & m, k, lg)],
                         u[cidx(i, j, (k + 1) & m, lg)], u[cidx(i, j, (k - 1) & m, lg)], f[c], kc);
    u[c] = uc + du;
}

// 1/x for finite non-zero x: hardware reciprocal refined by two Newton steps.
__device__ __forceinline__ double recip(double x)
{
    double y = __builtin_amdgcn_rcp(x);
    double e = fma(-x, y, 1.0);
    y = fma(y, e, y);
    e = fma(-x, y, 1.0);
    return fma(y, e, y);
}

// Newton-Gauss-Seidel step from precomputed exponentials: ec = e^{u_c},
// em = e^{-q u_c} - 1, neighbour values n* and their exponentials e*.  em is
// expm1_64's in every sweep: for n = 1 rsqrt(ec) - 1 would be cheaper (sweeps back to
// back, 512^3: 705 us for 727, 256^3: 92 for 98), but cancels for small u (solves of contrast 1e-6 stop
// at a residual of 2e-9) and is infinite where e^u underflows.
__device__ __forceinline__ double ngs_step_e(double uc, double ec, double em, double n0, double e0, double n1,
                                             double e1, double n2, double e2, double n3, double e3, double n4,
                                             double e4, double n5, double e5, double f, const OpConst &k)
{
    double d0 = n0 - uc, d1 = n1 - uc, d2 = n2 - uc, d3 = n3 - uc, d4 = n4 - uc, d5 = n5 - uc;
    double S1 = ((d0 + d1) + (d2 + d3)) + (d4 + d5);
    double S2 = ((e0 + e1) + (e2 + e3)) + (e4 + e5);
    double S3 = ((e0 * d0 + e1 * d1) + (e2 * d2 + e3 * d3)) + (e4 * d4 + e5 * d5);
    double L = k.ih2 * 0.5 * (S3 + ec * S1) + k.bC * em;
    double J = k.ih2 * 0.5 * (ec * (S1 - 6.0) - S2) - k.bC * k.q * (1.0 + em);
    double du = -(L - f) * recip(J);
    if (k.max_du > 0.0) du = fmin(fmax(du, -k.max_du), k.max_du);
    return du;
}

// One full red-black sweep, out of place: out = sweep(u), on levels with N >= 64
// (by default from 128^3 on).
//
// A workgroup has 15 waves, one per row of 128 cells (lane l: the pair
// k0 + 2 l, k0 + 2 l + 1), and marches along i.  In step p it updates the red
// cells of plane p + 1 and the black cells of plane p - 1.  The two updates of a
// lane do not depend on each other, which is why the black one trails by two
// planes: with one barrier per step and four waves per SIMD the dependent chain
// of an update is what a step would otherwise wait for.  Rows 1..13 are
// stored; rows 0 and 14 update only their red cells, which the black cells of
// rows 1 and 13 need (their outer neighbour is one more value per lane).  The
// red cells k0 - 1 and k0 + 128 of all rows are a sixteenth wave's.  A cell is
// kept as (u, e^u): e^u is evaluated when its plane is loaded and after its red
// update.  In every plane the updated column of a wave is uniform, so nothing
// is selected per lane.  LDS holds the old black cells of plane p + 1 and the
// new red cells of plane p - 1 (two buffers each, 63 KB).  Meshes narrower than
// a tile (N = 64) hold it twice: both copies of a cell get the same value.
//
// Bound: the float64 vector pipe and the latency of a step (one workgroup per
// CU: 128 registers).  Within a solve 0.71 ms per sweep of 512^3 (24 B per cell),
// 91 us of 256^3, 20 us of 128^3; a version with a row pair per thread, 12 x 60 of each 16 x 64 tile
// stored and a select for every operand issued twice the instructions: 1206 and
// 207 us.  What mattered besides: no spilled register (a scratch load waits for
// every prefetch before it), and exponentials after the barrier, not before it.
struct RowArgs {
    const double *u, *f;
    double *out;
    int lg, chunk;
    unsigned nkt, njt;
    OpConst kc;
};

typedef double2 RowLds[2][kRowF][kRowS];

__device__ __forceinline__ double row_update(const double2 &c, const double2 &n0, const double2 &n1, const double2 &n2,
                                             const double2 &n3, const double2 &n4, const double2 &n5, double f,
                                             const OpConst &kc)
{
    return c.x + ngs_step_e(c.x, c.y, expm1_64(-kc.q * c.x, kc.tab), n0.x, n0.y, n1.x, n1.y, n2.x, n2.y, n3.x,
                            n3.y, n4.x, n4.y, n5.x, n5.y, f, kc);
}

// S0: red column of the wave's row on plane i0 - 1.  RING: an outer row.
template <int S0, bool RING>
__device__ __forceinline__ void sweep_rows(const RowArgs &A, int i0, int j0, int k0, int row, int lane, RowLds &sO,
                                           RowLds &sN)
{
    const int lg = A.lg, m = (1 << lg) - 1;
    const int i1 = min(i0 + A.chunk, m + 1);
    const size_t plane = (size_t)1 << (2 * lg);
    const uint32_t pbytes = 8u << (2 * lg);
    const int jg = (j0 - 1 + row) & m;
    const bool stored = !RING && j0 - 1 + row <= m;  // uniform over the wave
    // byte offsets within a plane: the lane's pair, and (RING) the same in the row beyond
    const uint32_t kk = (uint32_t)((k0 + 2 * lane) & m);
    const uint32_t off = 8u * (((uint32_t)jg << lg) + kk);
    const uint32_t offo = 8u * (((uint32_t)((row == 0 ? jg - 1 : jg + 1) & m) << lg) + kk);
    auto pu = [&](int pl) { return PlaneBuf(A.u + (size_t)(pl & m) * plane, pbytes); };
    auto pf = [&](int pl) { return PlaneBuf(A.f + (size_t)(pl & m) * plane, pbytes); };
    const OpConst &kc = A.kc;
    auto cell = [&](double u) { return make_double2(u, exp64(u, kc.tab)); };
    // raw values of step p, two steps ahead: u of plane p + 2, f of plane p + 1;
    // RING: f of the red cell alone and its outer neighbour (column S), plane p + 1
    struct Raw {
        double2 u, f;
    };
    auto load = [&](int p, int S) {
        Raw w;
        w.u = pu(p + 2).ld2(off);
        if constexpr (RING)
            w.f = make_double2(pf(p + 1).ld(off + 8u * S), pu(p + 1).ld(offo + 8u * S));
        else
            w.f = pf(p + 1).ld2(off);
        return w;
    };
    // planes p - 1 (red new), p (red new) and p + 1 (old) of the pair; red cell of plane p - 2
    double2 A1[2], C0[2], C1[2], R2;
    double fb0 = 0.0, fb1 = 0.0;  // f of the black cells of planes p - 1 and p
    {
        const double2 u0 = pu(i0 - 2).ld2(off), u1 = pu(i0 - 1).ld2(off);
        C0[0] = cell(u0.x);
        C0[1] = cell(u0.y);
        C1[0] = cell(u1.x);
        C1[1] = cell(u1.y);
        A1[0] = A1[1] = R2 = C0[0];
    }
    Raw ra = load(i0 - 2, S0), rb = load(i0 - 1, 1 - S0);
    int buf = 0;
    auto step = [&](int p, auto Sc, Raw &raw) {
        constexpr int S = decltype(Sc)::value, T = 1 - S;
        double2(*O)[kRowS] = sO[buf], (*R)[kRowS] = sN[buf];
        O[row][lane + 1] = C1[T];
        R[row][lane + 1] = A1[S];
        __syncthreads();
        const double2 Q[2] = {cell(raw.u.x), cell(raw.u.y)};
        const double2 fv = raw.f;
        raw = load(p + 2, S);
        // red cell of plane p + 1
        double2 up, dn;
        if constexpr (RING) {
            const double2 o = cell(fv.y), in = O[row == 0 ? 1 : row - 1][lane + 1];
            up = make_double2(row == 0 ? o.x : in.x, row == 0 ? o.y : in.y);
            dn = make_double2(row == 0 ? in.x : o.x, row == 0 ? in.y : o.y);
        } else {
            up = O[row - 1][lane + 1];
            dn = O[row + 1][lane + 1];
        }
        const double ur = row_update(C1[S], Q[S], C0[S], dn, up, C1[T], O[row][S ? lane + 2 : lane],
                                         RING || !S ? fv.x : fv.y, kc);
        // black cell of plane p - 1
        if constexpr (!RING) {
            if (stored && p - 1 >= i0) {
                const double ub = row_update(A1[T], C0[T], R2, R[row + 1][lane + 1], R[row - 1][lane + 1], A1[S],
                                                 R[row][T ? lane + 2 : lane], fb0, kc);
                PlaneBuf(A.out + (size_t)(p - 1) * plane, pbytes)
                    .st2(off, S ? make_double2(ub, A1[1].x) : make_double2(A1[0].x, ub));
            }
        }
        R2 = A1[S];
        A1[0] = C0[0];
        A1[1] = C0[1];
        C0[T] = C1[T];
        C0[S] = cell(ur);
        C1[0] = Q[0];
        C1[1] = Q[1];
        fb0 = fb1;
        fb1 = S ? fv.x : fv.y;
        buf ^= 1;
    };
    for (int p = i0 - 2; p <= i1; p += 2) {
        step(p, std::integral_constant<int, S0>{}, ra);
        if (p < i1) step(p + 1, std::integral_constant<int, 1 - S0>{}, rb);
    }
}

// The red cells k0 - 1 (lanes 0..14, row = lane) and k0 + 128 (lanes 16..30) of
// the workgroup's rows, on the same steps: a cell is black and red in turn along
// i; black, its old value is published beside its row's black cells, red, it is
// updated and its new value published with the row's red ones.
__device__ __forceinline__ void sweep_ends(const RowArgs &A, int i0, int j0, int k0, int lane, RowLds &sO, RowLds &sN)
{
    const int lg = A.lg, m = (1 << lg) - 1;
    const int i1 = min(i0 + A.chunk, m + 1);
    const size_t plane = (size_t)1 << (2 * lg);
    const uint32_t pbytes = 8u << (2 * lg);
    const bool low = (lane & 16) == 0, live = (lane & 15) < kRowF && lane < 32;
    const int q = min(lane & 15, kRowF - 1), slot = low ? 0 : kRowS - 1, in = low ? 1 : kRowS - 2;
    const int j = (j0 - 1 + q) & m, k = (low ? k0 - 1 : k0 + kRowW) & m, k2 = (low ? k0 - 2 : k0 + kRowW + 1) & m;
    const uint32_t off = 8u * (((uint32_t)j << lg) + (uint32_t)k), off2 = 8u * (((uint32_t)j << lg) + (uint32_t)k2);
    const int jup = q > 0 ? q - 1 : 0, jdn = q < kRowF - 1 ? q + 1 : q;
    auto pu = [&](int pl) { return PlaneBuf(A.u + (size_t)(pl & m) * plane, pbytes); };
    auto pf = [&](int pl) { return PlaneBuf(A.f + (size_t)(pl & m) * plane, pbytes); };
    const OpConst &kc = A.kc;
    auto cell = [&](double u) { return make_double2(u, exp64(u, kc.tab)); };
    struct Raw {  // step p: u of plane p + 2; f and the outer neighbour of plane p + 1
        double u, f, u2;
    };
    auto load = [&](int p) { return Raw{pu(p + 2).ld(off), pf(p + 1).ld(off), pu(p + 1).ld(off2)}; };
    // the cell on planes p - 1, p, p + 1
    double2 h0 = cell(pu(i0 - 2).ld(off)), h1 = cell(pu(i0 - 1).ld(off)), hm = h0;
    Raw ra = load(i0 - 2), rb = load(i0 - 1);
    int buf = 0;
    auto step = [&](int p, Raw &raw) {
        const bool red = ((p + 1 + j + k) & 1) == 0;  // on planes p + 1 and p - 1
        double2(*O)[kRowS] = sO[buf], (*R)[kRowS] = sN[buf];
        const double2 hv = make_double2(red ? hm.x : h1.x, red ? hm.y : h1.y);
        if (live) (red ? R : O)[q][slot] = hv;
        __syncthreads();
        const double2 hn = cell(raw.u);
        const Raw cur = raw;
        raw = load(p + 2);
        if (live && red)
            h1 = cell(row_update(h1, hn, h0, O[jdn][slot], O[jup][slot], O[q][in], cell(cur.u2), cur.f, kc));
        hm = h0;
        h0 = h1;
        h1 = hn;
        buf ^= 1;
    };
    for (int p = i0 - 2; p <= i1; p += 2) {
        step(p, ra);
        if (p < i1) step(p + 1, rb);
    }
}

// grid: nkt njt ceil(N / chunk) workgroups; those of one XCD (blocks b, b + 8,
// ...) take consecutive tiles in j, which share their outer rows in its L2
__global__ __launch_bounds__(64 * (kRowF + 1)) void k_sweep_rows(RowArgs A)
{
    __shared__ RowLds sO, sN;
    MGFR_EXP_TABLE_TO_LDS(A.kc);
    const unsigned nb = gridDim.x, x = blockIdx.x & 7u, per = nb >> 3, rem = nb & 7u;
    const unsigned L = x * per + min(x, rem) + (blockIdx.x >> 3);
    const int kt = (int)(L % A.nkt), jt = (int)((L / A.nkt) % A.njt), it = (int)(L / (A.nkt * A.njt));
    const int k0 = kt * kRowW, j0 = jt * kRowI, i0 = it * A.chunk;
    const int row = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    const int s0 = (i0 - 1 + j0 - 1 + row) & 1;  // red column of the row on plane i0 - 1
    if (row == kRowF)
        sweep_ends(A, i0, j0, k0, lane, sO, sN);
    else if (row == 0 || row == kRowF - 1) {
        if (s0)
            sweep_rows<1, true>(A, i0, j0, k0, row, lane, sO, sN);
        else
            sweep_rows<0, true>(A, i0, j0, k0, row, lane, sO, sN);
    } else {
        if (s0)
            sweep_rows<1, false>(A, i0, j0, k0, row, lane, sO, sN);
        else
            sweep_rows<0, false>(A, i0, j0, k0, row, lane, sO, sN);
    }
}

// --------------------------------------------------------------- grid kernels

__global__ __launch_bounds__(kBlock) void k_sweep_half(double *__restrict__ u, const double *__restrict__ f,
                                                         int lg, int colour, OpConst kc)
{
    MGFR_EXP_TABLE_TO_LDS(kc);
    size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x;
    sweep_cell(u, f, t, lg, colour, kc);
}

// rbar -> fc, R u -> ubar_c
__global__ __launch_bounds__(kBlock) void k_residual_restrict(const double *__restrict__ u,
                                                                const double *__restrict__ f, int lg,
                                                                OpConst kc, double *__restrict__ ubar_c,
                                                                double *__restrict__ f_c)
{
    MGFR_EXP_TABLE_TO_LDS(kc);
    const int lgc = lg - 1;
    size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x;
    int K = (int)(t & ((1u << lgc) - 1));
    int J = (int)((t >> lgc) & ((1u << lgc) - 1));
    int I = (int)(t >> (2 * lgc));
    BlockRes br;
    block_residuals(u, f, I, J, K, lg, kc, br);
    ubar_c[t] = br.umean;
    f_c[t] = br.rmean;
}

// f_c += L_c(ubar), u_c = ubar
__global__ __launch_bounds__(kBlock) void k_coarse_rhs(const double *__restrict__ ubar, int lg, OpConst kc,
                                                         double *__restrict__ fc, double *__restrict__ uc)
{
    MGFR_EXP_TABLE_TO_LDS(kc);
    size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x;
    const int m = (1 << lg) - 1;
    int k = (int)(t & m), j = (int)((t >> lg) & m), i = (int)(t >> (2 * lg));
    fc[t] += op_at(ubar, i, j, k, lg, kc);
    uc[t] = ubar[t];
}

// one thread per coarse cell: its 8 daughters of the 2^lg mesh
__global__ __launch_bounds__(kBlock) void k_prolong_add(double *__restrict__ u, const double *__restrict__ uc,
                                                          const double *__restrict__ ub, int lg, int mode)
{
    const int lgc = lg - 1;
    const size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x;
    const int K = (int)(t & ((1u << lgc) - 1)), J = (int)((t >> lgc) & ((1u << lgc) - 1)), I = (int)(t >> (2 * lgc));
    prolong_block(u, uc, ub, I, J, K, lgc, mode);
}

template <int BS>
__device__ __forceinline__ void block_reduce_max_sum(double &mx, double &sm, double *sh)
{
    for (int o = 32; o > 0; o >>= 1) {
        mx = nanmax(mx, __shfl_xor(mx, o, 64));
        sm += __shfl_xor(sm, o, 64);
    }
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane == 0) {
        sh[w] = mx;
        sh[BS / 64 + w] = sm;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < BS / 64; ++i) {
            mx = nanmax(mx, sh[i]);
            sm += sh[BS / 64 + i];
        }
    }
}

// per-block max |r| and sum r^2 over the fine level (thread per 2x2x2 block)
__global__ __launch_bounds__(kBlock) void k_residual_norm(const double *__restrict__ u,
                                                            const double *__restrict__ f, int lg, OpConst kc,
                                                            double *__restrict__ partial, int nparts)
{
    MGFR_EXP_TABLE_TO_LDS(kc);
    __shared__ double sh[2 * kBlock / 64];
    const int lgc = lg - 1;
    const size_t nblk = (size_t)1 << (3 * lgc);
    double mx = 0.0, sm = 0.0;
    for (size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x; t < nblk; t += (size_t)gridDim.x * kBlock) {
        int K = (int)(t & ((1u << lgc) - 1));
        int J = (int)((t >> lgc) & ((1u << lgc) - 1));
        int I = (int)(t >> (2 * lgc));
        BlockRes br;
        block_residuals(u, f, I, J, K, lg, kc, br);
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            mx = nanmax(mx, fabs(br.r[c]));
            sm += br.r[c] * br.r[c];
        }
    }
    block_reduce_max_sum<kBlock>(mx, sm, sh);
    if (threadIdx.x == 0) {
        partial[blockIdx.x] = mx;
        partial[nparts + blockIdx.x] = sm;
    }
}

// The same for N >= 128, one exponential per cell: a workgroup marches over `chunk`
// planes of a tile of 14 rows of 128 cells and a row on either side, a row per wave,
// two cells per lane.  Neighbours in i are the planes before and after, in registers;
// those in j and k come from the plane's (u, e^u) in LDS (even cells before odd ones,
// the cells beyond the row's ends loaded by its first and last lane); loads run two
// planes ahead.  512^3: 0.67 ms (32 exponentials per 8 cells) -> 0.58; 256^3: 84 us -> 76.
__global__ __launch_bounds__(1024) void k_residual_norm_rows(const double *__restrict__ u, const double *__restrict__ f,
                                                             int lg, int chunk, unsigned nkt, unsigned njt, OpConst kc,
                                                             double *__restrict__ partial, int nparts)
{
    constexpr int W = 132;
    __shared__ double2 B[2][16][W];
    __shared__ double sh[2 * 1024 / 64];
    MGFR_EXP_TABLE_TO_LDS(kc);
    const int N = 1 << lg, M = N - 1;
    const unsigned nb = gridDim.x, x = blockIdx.x & 7u, per = nb >> 3, rem = nb & 7u;
    const unsigned L = x * per + min(x, rem) + (blockIdx.x >> 3);
    const int kt = (int)(L % nkt), jt = (int)((L / nkt) % njt), it = (int)(L / (nkt * njt));
    const int k0 = kt * kRowW, j0 = jt * 14, i0 = it * chunk, i1 = min(i0 + chunk, N);
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const bool own = w >= 1 && w <= 14 && j0 + w - 1 < N;
    const int jg = (j0 + w - 1) & M;
    const int ke = lane == 0 ? (k0 - 1) & M : lane == 63 ? (k0 + kRowW) & M : k0 + 2 * lane;
    const uint32_t oc = 8u * (uint32_t)((jg << lg) + k0 + 2 * lane), oe = 8u * (uint32_t)((jg << lg) + ke);
    const uint32_t bytes = 8u << (2 * lg);
    auto plane = [&](const double *a, int p) { return PlaneBuf(a + ((size_t)(p & M) << (2 * lg)), bytes); };
    auto slot = [](int k) { return (k & 1) * 66 + (k >> 1) + 1; };  // k = -1 .. 128
    double2 c0, c1, p0, p1;  // (u, e^u) of the two cells on this plane and the one before
    {
        const double2 a = plane(u, i0 - 1).ld2(oc), b = plane(u, i0).ld2(oc);
        p0 = make_double2(a.x, exp64(a.x, kc.tab));
        p1 = make_double2(a.y, exp64(a.y, kc.tab));
        c0 = make_double2(b.x, exp64(b.x, kc.tab));
        c1 = make_double2(b.y, exp64(b.y, kc.tab));
    }
    double ce = plane(u, i0).ld(oe);
    double2 un = plane(u, i0 + 1).ld2(oc), fc = plane(f, i0).ld2(oc);
    double xn = plane(u, i0 + 1).ld(oe);
    double mx = 0.0, sm = 0.0;
    int buf = 0;
    for (int p = i0; p < i1; ++p, buf ^= 1) {
        const int pn = min(p + 2, i1);  // the last plane needed is i1
        const double2 u2 = plane(u, pn).ld2(oc), f2 = plane(f, min(p + 1, i1 - 1)).ld2(oc);
        const double x2 = plane(u, pn).ld(oe);
        double2 *R = B[buf][w];
        R[slot(2 * lane)] = c0;
        R[slot(2 * lane + 1)] = c1;
        if (lane == 0 || lane == 63) R[slot(lane ? 128 : -1)] = make_double2(ce, exp64(ce, kc.tab));
        const double2 n0 = make_double2(un.x, exp64(un.x, kc.tab)), n1 = make_double2(un.y, exp64(un.y, kc.tab));
        __syncthreads();
        if (own) {
            const double2 *U = B[buf][w - 1], *D = B[buf][w + 1];
            auto res = [&](const double2 &c, const double2 &a, const double2 &b, const double2 &d, const double2 &e,
                           const double2 &l, const double2 &r, double fv) {
                const double d0 = a.x - c.x, d1 = b.x - c.x, d2 = d.x - c.x, d3 = e.x - c.x, d4 = r.x - c.x,
                             d5 = l.x - c.x;
                const double S1 = ((d0 + d1) + (d2 + d3)) + (d4 + d5);
                const double S3 = ((a.y * d0 + b.y * d1) + (d.y * d2 + e.y * d3)) + (r.y * d4 + l.y * d5);
                const double v = fv - (kc.ih2 * 0.5 * (S3 + c.y * S1) + kc.bC * expm1_64(-kc.q * c.x, kc.tab));
                mx = nanmax(mx, fabs(v));
                sm += v * v;
            };
            res(c0, n0, p0, D[slot(2 * lane)], U[slot(2 * lane)], R[slot(2 * lane - 1)], c1, fc.x);
            res(c1, n1, p1, D[slot(2 * lane + 1)], U[slot(2 * lane + 1)], c0, R[slot(2 * lane + 2)], fc.y);
        }
        p0 = c0;
        p1 = c1;
        c0 = n0;
        c1 = n1;
        ce = xn;
        un = u2;
        xn = x2;
        fc = f2;
    }
    __syncthreads();
    block_reduce_max_sum<1024>(mx, sm, sh);
    if (threadIdx.x == 0) {
        partial[blockIdx.x] = mx;
        partial[nparts + blockIdx.x] = sm;
    }
}

__global__ __launch_bounds__(kBlock) void k_residual_field(const double *__restrict__ u,
                                                             const double *__restrict__ f, int lg, OpConst kc,
                                                             double *__restrict__ r)
{
    MGFR_EXP_TABLE_TO_LDS(kc);
    size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x;
    const int m = (1 << lg) - 1;
    int k = (int)(t & m), j = (int)((t >> lg) & m), i = (int)(t >> (2 * lg));
    r[t] = f[t] - op_at(u, i, j, k, lg, kc);
}

// final reduction of nparts partials -> out[0] = max, out[1] = sum
__global__ __launch_bounds__(1024) void k_final_reduce(const double *__restrict__ partial, int nparts,
                                                        double *__restrict__ out)
{
    __shared__ double sh[2 * 1024 / 64];
    double mx = 0.0, sm = 0.0;
    for (int i = threadIdx.x; i < nparts; i += 1024) {
        mx = nanmax(mx, partial[i]);
        sm += partial[nparts + i];
    }
    block_reduce_max_sum<1024>(mx, sm, sh);
    if (threadIdx.x == 0) {
        out[0] = mx;
        out[1] = sm;
    }
}

// f = s * delta with per-block max |f| partials
__global__ __launch_bounds__(kBlock) void k_source(const double *__restrict__ delta, double s, size_t n,
                                                     double *__restrict__ f, double *__restrict__ partial,
                                                     int nparts)
{
    __shared__ double sh[2 * kBlock / 64];
    double mx = 0.0, sm = 0.0;
    for (size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x; t < n; t += (size_t)gridDim.x * kBlock) {
        double v = s * delta[t];
        f[t] = v;
        mx = nanmax(mx, fabs(v));
    }
    block_reduce_max_sum<kBlock>(mx, sm, sh);
    if (threadIdx.x == 0) {
        partial[blockIdx.x] = mx;
        partial[nparts + blockIdx.x] = 0.0;
    }
}

// Screened-limit initial guess: u = -(n+1) log1p(s max(delta, 0)) with
// s = Omega_m a^-3 / C(a) (the local balance of the field equation where the
// Laplacian term is negligible).
__global__ __launch_bounds__(kBlock) void k_screened_guess(const double *__restrict__ delta, double s,
                                                             double np1, size_t n, double *__restrict__ u)
{
    for (size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x; t < n; t += (size_t)gridDim.x * kBlock) {
        const double d = delta[t];
        u[t] = -np1 * log1p(s * (d > 0.0 ? d : 0.0));
    }
}

// delta_eff = delta/3 - c expm1(-q u) with c = C / (3 Omega_m a^-3)
__global__ __launch_bounds__(kBlock) void k_effective_density(const double *__restrict__ delta,
                                                                const double *__restrict__ u, double c, double q,
                                                                size_t n, double *__restrict__ out)
{
    for (size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x; t < n; t += (size_t)gridDim.x * kBlock)
        out[t] = delta[t] / 3.0 - c * expm1(-q * u[t]);
}

__global__ __launch_bounds__(kBlock) void k_dfr(const double *__restrict__ u, double fbar, size_t n,
                                                  double *__restrict__ dfr)
{
    for (size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x; t < n; t += (size_t)gridDim.x * kBlock)
        dfr[t] = -fbar * expm1(u[t]);
}

// ------------------------------------------------------------- tail kernel
// All levels with N <= kTailN inside one workgroup: the V-cycle from the 16^3
// (or 8^3) level down to the 4^3 grid and back.
//
// Bound: a serial chain of some 100 half-sweeps of few cells, so what counts
// is the latency of each.  Every level lives in LDS as (u, e^u) pairs, so that
// an update reads its neighbours' exponentials and evaluates one of its own
// (in global memory, with eight exponentials and a division per update, the
// cycle took 137 us for V(2,2) and 192 us for V(4,4); now 44 and 60 us).  A
// thread owns W consecutive cells of a row (TailGrid) and keeps their values
// and f in registers through a smoothing phase.

struct TailArgs {
    double *u;        // top level, in and out
    const double *f;
    double ih2[3];    // 16^3, 8^3, 4^3
    int lg0;          // 4 or 3
    int pre, post, coarse, mode;
    double bC, q, max_du;
    const double *tab;  // exponential's table (the kernel points it at its LDS copy)
};

template <int LG>
struct TailLevel : TailGrid<LG> {
    double2 *ue;  // (u, e^u)
    double *f, *ub;
};

__device__ __forceinline__ double2 tail_update(double2 c, double2 n0, double2 n1, double2 n2, double2 n3, double2 n4,
                                               double2 n5, double f, const OpConst &kc)
{
    const double un = c.x + ngs_step_e(c.x, c.y, expm1_64(-kc.q * c.x, kc.tab), n0.x, n0.y, n1.x, n1.y, n2.x, n2.y,
                                       n3.x, n3.y, n4.x, n4.y, n5.x, n5.y, f, kc);
    return make_double2(un, exp64(un, kc.tab));
}

// Red-black sweeps of the 16^3 or 8^3 level.
template <int LG>
__device__ __forceinline__ void tail_sweeps(const TailLevel<LG> &T, int sweeps, const OpConst &kc)
{
    using L = TailLevel<LG>;
    constexpr int W = L::W, M = L::M;
    const int t = threadIdx.x;
    const bool own = t < L::THREADS;
    int i = 0, j = 0, k0 = 0;
    double2 x[W];
    double f[W];
    if (own) {
        L::cell(t, i, j, k0);
#pragma unroll
        for (int c = 0; c < W; ++c) {
            x[c] = T.ue[L::slot(i, j, k0 + c)];
            f[c] = T.f[L::slot(i, j, k0 + c)];
        }
    }
    const int par = __builtin_amdgcn_readfirstlane((i + j) & 1);  // uniform over the wave
    const int ip = (i + 1) & M, im = (i - 1) & M, jp = (j + 1) & M, jm = (j - 1) & M;
    // update columns B, B + 2, ... of the thread's cells
    auto half = [&](auto Bc) {
        constexpr int B = decltype(Bc)::value;
        const double2 out = T.ue[L::slot(i, j, B ? (k0 + W) & M : (k0 - 1) & M)];
        double2 y[W];
#pragma unroll
        for (int c = B; c < W; c += 2) {
            const int k = k0 + c;
            const double2 l = c == 0 ? out : x[c - 1], r = c == W - 1 ? out : x[(c + 1) % W];
            y[c] = tail_update(x[c], T.ue[L::slot(ip, j, k)], T.ue[L::slot(im, j, k)], T.ue[L::slot(i, jp, k)],
                                       T.ue[L::slot(i, jm, k)], r, l, f[c], kc);
        }
#pragma unroll
        for (int c = B; c < W; c += 2) {
            x[c] = y[c];
            T.ue[L::slot(i, j, k0 + c)] = y[c];
        }
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
__device__ __forceinline__ void tail_sweeps4(const TailLevel<2> &T, int sweeps, const OpConst &kc)
{
    using L = TailLevel<2>;
    if (threadIdx.x < 64) {
        int i, j, k;
        L::cell(threadIdx.x, i, j, k);
        const int c = L::slot(i, j, k), par = (i + j + k) & 1;
        const int n0 = L::slot((i + 1) & 3, j, k), n1 = L::slot((i - 1) & 3, j, k), n2 = L::slot(i, (j + 1) & 3, k),
                  n3 = L::slot(i, (j - 1) & 3, k), n4 = L::slot(i, j, (k + 1) & 3), n5 = L::slot(i, j, (k - 1) & 3);
        double2 x = T.ue[c];
        const double f = T.f[c];
        for (int h = 0; h < 2 * sweeps; ++h) {
            if (par == (h & 1)) {
                x = tail_update(x, T.ue[n0], T.ue[n1], T.ue[n2], T.ue[n3], T.ue[n4], T.ue[n5], f, kc);
                T.ue[c] = x;
            }
            wave_lds_sync();
        }
    }
    __syncthreads();
}

// L(u) at a cell of a tail level
template <int LG>
__device__ __forceinline__ double tail_op(const TailLevel<LG> &T, int i, int j, int k, double2 c, const OpConst &kc)
{
    using L = TailLevel<LG>;
    constexpr int M = L::M;
    const double2 n0 = T.ue[L::slot((i + 1) & M, j, k)], n1 = T.ue[L::slot((i - 1) & M, j, k)],
                  n2 = T.ue[L::slot(i, (j + 1) & M, k)], n3 = T.ue[L::slot(i, (j - 1) & M, k)],
                  n4 = T.ue[L::slot(i, j, (k + 1) & M)], n5 = T.ue[L::slot(i, j, (k - 1) & M)];
    const double d0 = n0.x - c.x, d1 = n1.x - c.x, d2 = n2.x - c.x, d3 = n3.x - c.x, d4 = n4.x - c.x, d5 = n5.x - c.x;
    const double S1 = ((d0 + d1) + (d2 + d3)) + (d4 + d5);
    const double S3 = ((n0.y * d0 + n1.y * d1) + (n2.y * d2 + n3.y * d3)) + (n4.y * d4 + n5.y * d5);
    return kc.ih2 * 0.5 * (S3 + c.y * S1) + kc.bC * expm1_64(-kc.q * c.x, kc.tab);
}

// Restriction to the next level: means of u and of the residual over the eight
// daughters, then the coarse source f_c = L_c(R u) + R(f - L u), u_c = R u.
template <int LG>
__device__ __forceinline__ void tail_restrict(const TailLevel<LG> &T, const TailLevel<LG - 1> &C, const OpConst &kf,
                                              const OpConst &kcc)
{
    using L = TailLevel<LG>;
    using LC = TailLevel<LG - 1>;
    const int t = threadIdx.x;
    const int I = t >> (2 * LG - 2), J = (t >> (LG - 1)) & LC::M, K = t & LC::M;
    double r = 0.0, ub = 0.0;
    if (t < LC::CELLS) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int i = 2 * I + (e >> 2), j = 2 * J + ((e >> 1) & 1), k = 2 * K + (e & 1), c = L::slot(i, j, k);
            const double2 x = T.ue[c];
            ub += x.x;
            r += T.f[c] - tail_op(T, i, j, k, x, kf);
        }
        ub *= 0.125;
        r *= 0.125;
        const int c = LC::slot(I, J, K);
        C.ub[c] = ub;
        C.ue[c] = make_double2(ub, exp64(ub, kf.tab));
    }
    __syncthreads();
    if (t < LC::CELLS) {
        const int c = LC::slot(I, J, K);
        C.f[c] = r + tail_op(C, I, J, K, C.ue[c], kcc);
    }
    __syncthreads();
}

// u += P(u_c - R u): the thread's cells from their W / 2 parents
template <int LG>
__device__ __forceinline__ void tail_prolong(const TailLevel<LG> &T, const TailLevel<LG - 1> &C, int mode,
                                             const double *tab)
{
    using L = TailLevel<LG>;
    using LC = TailLevel<LG - 1>;
    constexpr int MC = LC::M;
    if (threadIdx.x < L::THREADS) {
        int i, j, k0;
        L::cell(threadIdx.x, i, j, k0);
        auto d = [&](int a, int b, int c) {
            const int s = LC::slot(a & MC, b & MC, c & MC);
            return C.ue[s].x - C.ub[s];
        };
#pragma unroll
        for (int h = 0; h < L::W / 2; ++h) {
            const int I = i >> 1, J = j >> 1, K = (k0 >> 1) + h;
            double v0 = d(I, J, K), gz = 0.0;
            if (mode == 0) {
                v0 += ((i & 1) ? 0.125 : -0.125) * (d(I + 1, J, K) - d(I - 1, J, K));
                v0 += ((j & 1) ? 0.125 : -0.125) * (d(I, J + 1, K) - d(I, J - 1, K));
                gz = 0.125 * (d(I, J, K + 1) - d(I, J, K - 1));
            }
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int s = L::slot(i, j, k0 + 2 * h + c);
                const double u = T.ue[s].x + (c ? v0 + gz : v0 - gz);
                T.ue[s] = make_double2(u, exp64(u, tab));
            }
        }
    }
    __syncthreads();
}

__global__ __launch_bounds__(kTailThreads) void k_tail(TailArgs A)
{
    __shared__ double2 s_ue[4096 + 512 + 64];
    __shared__ double s_f[4096 + 512 + 64], s_ub[512 + 64], s_tab[64];
    const int t = threadIdx.x;
    if (t < 64) s_tab[t] = A.tab[t];
    const TailLevel<4> T4{{}, s_ue, s_f, nullptr};
    const TailLevel<3> T3{{}, s_ue + 4096, s_f + 4096, s_ub};
    const TailLevel<2> T2{{}, s_ue + 4608, s_f + 4608, s_ub + 512};
    const OpConst k4{A.ih2[0], A.bC, A.q, A.max_du, s_tab}, k3{A.ih2[1], A.bC, A.q, A.max_du, s_tab},
        k2{A.ih2[2], A.bC, A.q, A.max_du, s_tab};
    __syncthreads();
    const int lg = A.lg0, n0 = 1 << (3 * lg), m = (1 << lg) - 1;
    auto slot0 = [&](int c) {
        const int i = c >> (2 * lg), j = (c >> lg) & m, k = c & m;
        return lg == 4 ? TailLevel<4>::slot(i, j, k) : 4096 + TailLevel<3>::slot(i, j, k);
    };
    for (int c = t; c < n0; c += kTailThreads) {
        const double u = A.u[c];
        s_ue[slot0(c)] = make_double2(u, exp64(u, s_tab));
        s_f[slot0(c)] = A.f[c];
    }
    __syncthreads();
    if (lg == 4) {
        tail_sweeps(T4, A.pre, k4);
        tail_restrict(T4, T3, k4, k3);
    }
    tail_sweeps(T3, A.pre, k3);
    tail_restrict(T3, T2, k3, k2);
    tail_sweeps4(T2, A.coarse, k2);
    tail_prolong(T3, T2, A.mode, s_tab);
    tail_sweeps(T3, A.post, k3);
    if (lg == 4) {
        tail_prolong(T4, T3, A.mode, s_tab);
        tail_sweeps(T4, A.post, k4);
    }
    for (int c = t; c < n0; c += kTailThreads) A.u[c] = s_ue[slot0(c)].x;
}

// ------------------------------------------------------------ host launches

static inline unsigned nblocks(size_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

// ------------------------------------------------- small levels, several half-sweeps
//
// H half-sweeps (2: one red-black sweep, 4: two) of the 32^3 or 64^3 level in one
// launch, out of place.  A workgroup owns 4 x 4 rows of the mesh and holds them
// with H rows on every side in LDS as (u, e^u): each half-sweep updates one row
// less on every side, so that the cells of the tile end with the values that H
// launches of one colour each would give, and no workgroup waits for another.
// A row's even cells lie before its odd ones: the lanes of an access take
// consecutive 16-byte places.
// Bound: float64 arithmetic, the surrounding rows included (1.6 times the cells'
// updates for H = 2, 3.4 for H = 4), and the latency of a launch.  One launch per
// colour took 3.5-3.9 us and the gap to the next: 32^3, two sweeps 4 x 3.5 -> 7.3 us
// (H = 2 twice: 8.8); 64^3, one sweep 2 x 3.9 -> 5.3 us.
// PRO: the first sweeps after the coarse level: u + P(uc - ub) is formed as the tile
// is loaded (about 1 us more, against 4.8 us of a launch of its own).
template <int LG, int H, bool PRO>
__global__ __launch_bounds__(1024) void k_sweep_tile(const double *__restrict__ u, const double *__restrict__ f,
                                                     double *__restrict__ out, OpConst kc,
                                                     const double *__restrict__ uc, const double *__restrict__ ub,
                                                     int mode)
{
    using P = TileProlong<double, LG, 4 + 2 * H>;
    __shared__ double sd[PRO ? P::CELLS : 1];
    constexpr int N = 1 << LG, M = N - 1, E = 4 + 2 * H, HALF = N / 2, NT = 1024;
    __shared__ double2 ue[E * E * N];
    MGFR_EXP_TABLE_TO_LDS(kc);
    const int t = threadIdx.x;
    const int i0 = 4 * (int)(blockIdx.x / (N / 4)) - H, j0 = 4 * (int)(blockIdx.x % (N / 4)) - H;
    auto slot = [](int i, int j, int k) { return ((i * E + j) << LG) + (k & 1) * HALF + (k >> 1); };
    auto cell = [&](int i, int j, int k) {
        return ((((size_t)((i0 + i) & M) << LG) + (size_t)((j0 + j) & M)) << LG) + (size_t)k;
    };
    // the cell of thread t, round q, of half-sweep h: (4 + 2 m)^2 rows of N / 2 cells, m = H - 1 - h
    auto place = [&](int h, int q, int &i, int &j, int &k) {
        const int m = H - 1 - h, D = 4 + 2 * m, e = t + q * NT, row = e / HALF;
        i = H - m + row / D;
        j = H - m + row % D;
        k = 2 * (e % HALF) + ((i0 + i + j0 + j + h) & 1);
        return row < D * D;
    };
    constexpr int R = ((4 + 2 * (H - 1)) * (4 + 2 * (H - 1)) * HALF + NT - 1) / NT;  // rounds of the first half-sweep
    double fv[H][R];
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
        for (int q = 0; q < R; ++q) {
            int i, j, k;
            fv[h][q] = place(h, q, i, j, k) ? f[cell(i, j, k)] : 0.0;
        }
    constexpr int RL = (E * E * N + NT - 1) / NT;
    double x[RL];
#pragma unroll
    for (int q = 0; q < RL; ++q) {
        const int e = t + q * NT, r = e >> LG;
        x[q] = r < E * E ? u[cell(r / E, r % E, e & M)] : 0.0;
    }
    if constexpr (PRO) {
        P::template load<NT>(sd, uc, ub, i0, j0);
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < RL; ++q) {
        const int e = t + q * NT, r = e >> LG, k = e & M;
        if (r < E * E) {
            if (PRO) x[q] += P::value(sd, r / E, r % E, k, mode);
            ue[slot(r / E, r % E, k)] = make_double2(x[q], exp64(x[q], kc.tab));
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
                ue[c] = tail_update(ue[c], ue[c + E * N], ue[c - E * N], ue[c + N], ue[c - N],
                                            ue[side + (((k + 1) & M) >> 1)], ue[side + (((k - 1) & M) >> 1)], fv[h][q], kc);
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < (16 * N + NT - 1) / NT; ++q) {
        const int e = t + q * NT, r = e >> LG, k = e & M;
        if (r < 16) out[cell(H + (r >> 2), H + (r & 3), k)] = ue[slot(H + (r >> 2), H + (r & 3), k)].x;
    }
}

template <int LG, int H>
static void launch_tile(mgfr_ctx *c, Level &L, const double *f, const OpConst &kc, const Level *from)
{
    const unsigned nb = (unsigned)((L.N / 4) * (L.N / 4));
    const double *uc = from ? from->u : nullptr, *ub = from ? from->ubar : nullptr;
    auto go = [&](auto *k) { k<<<nb, 1024, 0, c->stream>>>(L.u, f, L.alt, kc, uc, ub, c->p.prolong); };
    from ? go(k_sweep_tile<LG, H, true>) : go(k_sweep_tile<LG, H, false>);
    std::swap(L.u, L.alt);
}

// 32^3 and 64^3, unless they run the fused sweep or one kernel per colour: see k_sweep_tile
static bool tile_level(const mgfr_ctx *c, const Level &L)
{
    return (L.N == 32 || L.N == 64) && c->fused_min_n > L.N && L.alt != nullptr;
}

static int timer_slot(mgfr_ctx *c, int *slot)
{
    Timer &T = c->sweep_timer;
    if (T.used + 2 > (int)T.ev.size()) {
        for (int e = 0; e < 16; ++e) {
            hipEvent_t ev;
            MGFR_HIP(hipEventCreate(&ev));
            T.ev.push_back(ev);
        }
    }
    *slot = T.used;
    T.used += 2;
    return MGFR_OK;
}

// Planes per workgroup of the fused sweeps: one workgroup runs on a CU at a time
// and spends chunk + 3 steps, so take the chunk with the fewest steps over all
// rounds of the 256 CUs.
int row_chunk(int N, unsigned cols)
{
    int best = N;
    long cost = -1;
    for (int n = 1; n <= N / 4; ++n) {
        const int chunk = (N + n - 1) / n;
        const long rounds = ((long)cols * ((N + chunk - 1) / chunk) + 255) / 256;
        const long c = rounds * (chunk + 3);
        if (cost < 0 || c < cost) {
            cost = c;
            best = chunk;
        }
    }
    return best;
}

// `sweeps` red-black sweeps on level l.  Levels with N >= fused_min_n use the
// out-of-place fused kernel, tile levels k_sweep_tile, and both swap L.u / L.alt
// after each launch; the others update L.u in place with one kernel per colour.
// With `from` (tile levels, at least one sweep) the correction of that coarser
// level is added first.
int launch_sweep64(mgfr_ctx *c, int l, double *u_unused, const double *f, int sweeps, bool timed, const Level *from)
{
    (void)u_unused;
    Level &L = c->lev[l];
    OpConst kc = level_const(c, l);
    const bool fused = c->fused_min_n > 0 && L.N >= c->fused_min_n && L.alt != nullptr;
    // Two sweeps in one launch on 32^3 (7.3 us against 8.8 for two launches, 64
    // workgroups), not on 64^3, whose 256 workgroups then redo more than the
    // launch saves (13.3 us against 11.8)
    const bool tile = tile_level(c, L);
    const size_t half = (size_t)1 << (3 * L.lg - 1);
    for (int s = 0; s < sweeps; ++s) {
        int slot = -1;
        if (timed) {
            int rc = timer_slot(c, &slot);
            if (rc) return rc;
            MGFR_HIP(hipEventRecord(c->sweep_timer.ev[slot], c->stream));
        }
        if (fused) {
            const unsigned nkt = (unsigned)std::max(1, L.N / kRowW), njt = (unsigned)((L.N + kRowI - 1) / kRowI);
            const int chunk = row_chunk(L.N, nkt * njt);
            const RowArgs A{L.u, f, L.alt, L.lg, chunk, nkt, njt, kc};
            const unsigned nb = nkt * njt * (unsigned)((L.N + chunk - 1) / chunk);
            k_sweep_rows<<<nb, 64 * (kRowF + 1), 0, c->stream>>>(A);
            std::swap(L.u, L.alt);
        } else if (tile) {
            if (L.N == 64) {
                launch_tile<6, 2>(c, L, f, kc, from);
            } else if (!timed && s + 1 < sweeps) {  // timing counts one sweep per launch
                launch_tile<5, 4>(c, L, f, kc, from);
                ++s;
            } else {
                launch_tile<5, 2>(c, L, f, kc, from);
            }
            from = nullptr;
        } else {
            for (int colour = 0; colour < 2; ++colour)
                k_sweep_half<<<nblocks(half), kBlock, 0, c->stream>>>(L.u, f, L.lg, colour, kc);
        }
        if (timed) MGFR_HIP(hipEventRecord(c->sweep_timer.ev[slot + 1], c->stream));
    }
    MGFR_HIP(hipGetLastError());
    return MGFR_OK;
}

static int launch_tail(mgfr_ctx *c, int l0)
{
    const Level &L = c->lev[l0];
    TailArgs A;
    A.u = L.u;
    A.f = L.f;
    A.lg0 = L.lg;  // 4 or 3: meshes have at least 8 cells a side
    for (int k = 0; k < 3; ++k) {
        const double h = c->p.box / (16 >> k);
        A.ih2[k] = 1.0 / (h * h);
    }
    A.pre = c->p.pre_smooth;
    A.post = c->p.post_smooth;
    A.coarse = c->p.coarse_sweeps;
    A.mode = c->p.prolong;
    A.bC = c->bC;
    A.q = c->q;
    A.max_du = c->p.max_du;
    A.tab = c->exp2tab;
    k_tail<<<1, kTailThreads, 0, c->stream>>>(A);
    MGFR_HIP(hipGetLastError());
    return MGFR_OK;
}

int vcycle64(mgfr_ctx *c, int l)
{
    Level &L = c->lev[l];
    if (L.N <= kTailN) return launch_tail(c, l);
    int rc;
    if ((rc = launch_sweep64(c, l, L.u, L.f, c->p.pre_smooth, l == 0 && c->timing))) return rc;
    Level &Lc = c->lev[l + 1];
    const size_t nc = (size_t)1 << (3 * Lc.lg);
    k_residual_restrict<<<nblocks(nc), kBlock, 0, c->stream>>>(L.u, L.f, L.lg, level_const(c, l), Lc.ubar, Lc.f);
    k_coarse_rhs<<<nblocks(nc), kBlock, 0, c->stream>>>(Lc.ubar, Lc.lg, level_const(c, l + 1), Lc.f, Lc.u);
    MGFR_HIP(hipGetLastError());
    if ((rc = vcycle64(c, l + 1))) return rc;
    const bool with_sweep = tile_level(c, L) && c->p.post_smooth > 0;
    if (!with_sweep) {
        k_prolong_add<<<nblocks(nc), kBlock, 0, c->stream>>>(L.u, Lc.u, Lc.ubar, L.lg, c->p.prolong);
        MGFR_HIP(hipGetLastError());
    }
    return launch_sweep64(c, l, L.u, L.f, c->p.post_smooth, l == 0 && c->timing, with_sweep ? &Lc : nullptr);
}

int launch_residual_norm64(mgfr_ctx *c, int l, const double *u, const double *f, double *rmax, double *rsumsq)
{
    Level &L = c->lev[l];
    const size_t nblk = (size_t)1 << (3 * (L.lg - 1));
    unsigned g = (unsigned)std::min<size_t>(nblocks(nblk), (size_t)c->nparts);
    // whole rows of 128 cells, and a partial per workgroup
    const unsigned nkt = (unsigned)std::max(1, L.N / kRowW), njt = (unsigned)((L.N + 13) / 14);
    const int chunk = L.N >= kRowW ? row_chunk(L.N, nkt * njt) : L.N;
    const unsigned gr = nkt * njt * (unsigned)((L.N + chunk - 1) / chunk);
    if (L.N >= kRowW && gr <= (unsigned)c->nparts) {
        g = gr;
        k_residual_norm_rows<<<g, 1024, 0, c->stream>>>(u, f, L.lg, chunk, nkt, njt, level_const(c, l), c->partial,
                                                        (int)g);
    } else {
        k_residual_norm<<<g, kBlock, 0, c->stream>>>(u, f, L.lg, level_const(c, l), c->partial, (int)g);
    }
    k_final_reduce<<<1, 1024, 0, c->stream>>>(c->partial, (int)g, c->dscal);
    MGFR_HIP(hipGetLastError());
    MGFR_HIP(hipMemcpyAsync(c->hscal, c->dscal, 2 * sizeof(double), hipMemcpyDeviceToHost, c->stream));
    MGFR_HIP(hipStreamSynchronize(c->stream));
    *rmax = c->hscal[0];
    *rsumsq = c->hscal[1];
    return MGFR_OK;
}

int collect_timing(mgfr_ctx *c, mgfr_stats *st)
{
    Timer &T = c->sweep_timer;
    for (int e = 0; e + 1 < T.used; e += 2) {
        float ms = 0;
        MGFR_HIP(hipEventElapsedTime(&ms, T.ev[e], T.ev[e + 1]));
        if (st) {
            st->t_sweep_ms += ms;
            st->n_sweep_launches += 1;
        }
    }
    T.used = 0;
    return MGFR_OK;
}

// ---------------------------------------------------------------- validation

static int validate(const mgfr_params *p)
{
    if (!p) return set_error(MGFR_ERR_ARG, "params is NULL");
    if (!(p->box > 0) || !std::isfinite(p->box)) return set_error(MGFR_ERR_ARG, "box must be > 0");
    if (!(p->a > 0) || !std::isfinite(p->a)) return set_error(MGFR_ERR_ARG, "a must be > 0");
    if (!(p->omega_m > 0)) return set_error(MGFR_ERR_ARG, "omega_m must be > 0");
    if (!(p->omega_l >= 0)) return set_error(MGFR_ERR_ARG, "omega_l must be >= 0");
    if (!(p->fr0_abs > 0) || !std::isfinite(p->fr0_abs)) return set_error(MGFR_ERR_ARG, "fr0_abs must be > 0");
    if (p->n < 1) return set_error(MGFR_ERR_ARG, "n must be >= 1");
    if (p->mesh < 8 || p->mesh > 1024 || (p->mesh & (p->mesh - 1)))
        return set_error(MGFR_ERR_ARG, "mesh must be a power of two in [8, 1024], got %d", p->mesh);
    if (p->refine_levels != 0) return set_error(MGFR_ERR_ARG, "refine_levels must be 0 for a uniform mesh");
    if (!(p->tol > 0)) return set_error(MGFR_ERR_ARG, "tol must be > 0");
    if (p->pre_smooth < 0 || p->post_smooth < 0) return set_error(MGFR_ERR_ARG, "smoothing counts must be >= 0");
    if (p->coarse_sweeps < 1) return set_error(MGFR_ERR_ARG, "coarse_sweeps must be >= 1");
    if (p->max_vcycles < 0) return set_error(MGFR_ERR_ARG, "max_vcycles must be >= 0");
    if (p->coarse_cycles < 0) return set_error(MGFR_ERR_ARG, "coarse_cycles must be >= 0");
    if (p->prolong != MGFR_PROLONG_LINEAR && p->prolong != MGFR_PROLONG_INJECT)
        return set_error(MGFR_ERR_ARG, "prolong must be 0 (linear) or 1 (injection)");
    if (p->precision != MGFR_FP64 && p->precision != MGFR_MIXED)
        return set_error(MGFR_ERR_ARG, "precision must be MGFR_FP64 or MGFR_MIXED");
    if (p->nn_mode != MGFR_NN_NONE && p->nn_mode != MGFR_NN_COARSE)
        return set_error(MGFR_ERR_ARG, "nn_mode must be MGFR_NN_NONE or MGFR_NN_COARSE");
    return MGFR_OK;
}

static void background(const mgfr_params *p, double *fbar, double *beta, double *C)
{
    // Sec. 2: R_bar = 3 H0^2 (Omega_m a^-3 + 4 Omega_L); fbar_R(a) = fbar_R0 (R_bar0/R_bar(a))^(n+1)
    double r = 4.0 * p->omega_l / p->omega_m;
    double a3 = 1.0 / (p->a * p->a * p->a);
    *fbar = p->fr0_abs * std::pow((1.0 + r) / (a3 + r), p->n + 1);
    *C = p->omega_m * a3 + 4.0 * p->omega_l;
    *beta = p->a * p->a / (kCOverH0 * kCOverH0) / *fbar;
}

}  // namespace mgfr

using namespace mgfr;

// ================================================================== C ABI

extern "C" const char *mgfr_last_error(void) { return g_err.c_str(); }

extern "C" int mgfr_background(const mgfr_params *p, double *fbar, double *beta, double *C)
{
    int rc = validate(p);
    if (rc) return rc;
    double a, b, c;
    background(p, &a, &b, &c);
    if (fbar) *fbar = a;
    if (beta) *beta = b;
    if (C) *C = c;
    return MGFR_OK;
}

static void free_ctx(mgfr_ctx *c)
{
    if (!c) return;
    nn_free(c);
    bin_free(c);
    pm_free(c);
    for (int l = 0; l < kMaxLevels; ++l) {
        Level &L = c->lev[l];
        if (l > 0) {
            (void)hipFree(L.u);
            (void)hipFree(L.alt);
        }
        (void)hipFree(L.f);
        (void)hipFree(L.ubar);
        (void)hipFree(L.e32);
        (void)hipFree(L.r32);
        (void)hipFree(L.u32);
        (void)hipFree(L.ebar32);
        (void)hipFree(L.e32alt);
    }
    (void)hipFree(c->alt0);
    (void)hipFree(c->partial);
    (void)hipFree(c->dscal);
    (void)hipFree(c->dflag);
    (void)hipFree(c->r64);
    (void)hipFree(c->exp2tab);
    if (c->hscal) (void)hipHostFree(c->hscal);
    for (hipEvent_t e : c->sweep_timer.ev) (void)hipEventDestroy(e);
    if (c->ev_a) (void)hipEventDestroy(c->ev_a);
    if (c->ev_b) (void)hipEventDestroy(c->ev_b);
    if (c->ev_c) (void)hipEventDestroy(c->ev_c);
    delete c;
}

static int create_impl(const mgfr_params *p, void *stream, mgfr_ctx *c)
{
    c->p = *p;
    c->stream = (hipStream_t)stream;
    MGFR_HIP(hipGetDevice(&c->device));
    background(p, &c->fbar, &c->beta, &c->C);
    c->bC = c->beta * c->C;
    c->q = 1.0 / (p->n + 1);
    int N = p->mesh, lg = 0;
    while ((1 << lg) < N) ++lg;
    c->nlev = 0;
    for (int n = N, l = 0; n >= 4; n /= 2, ++l) {
        Level &L = c->lev[l];
        L.N = n;
        L.lg = lg - l;
        L.h = p->box / n;
        size_t bytes = sizeof(double) * (size_t)n * n * n;
        MGFR_HIP(hipMalloc(&L.f, bytes));
        if (l > 0) {
            MGFR_HIP(hipMalloc(&L.u, bytes));
            MGFR_HIP(hipMalloc(&L.ubar, bytes));
        }
        if (n >= 32) {  // second buffer for out-of-place sweeps
            MGFR_HIP(hipMalloc(&L.alt, bytes));
            if (l == 0) c->alt0 = L.alt;
        }
        c->nlev = l + 1;
    }
    c->nparts = 4096;
    MGFR_HIP(hipMalloc(&c->partial, sizeof(double) * 2 * c->nparts));
    {
        double tab[64];
        for (int j = 0; j < 64; ++j) tab[j] = (double)exp2l((long double)j / 64.0L);
        MGFR_HIP(hipMalloc(&c->exp2tab, sizeof tab));
        MGFR_HIP(hipMemcpy(c->exp2tab, tab, sizeof tab, hipMemcpyHostToDevice));
    }
    MGFR_HIP(hipMalloc(&c->dscal, sizeof(double) * 8));
    MGFR_HIP(hipMalloc(&c->dflag, sizeof(int) * 4));
    MGFR_HIP(hipHostMalloc(&c->hscal, sizeof(double) * 8, hipHostMallocDefault));
    MGFR_HIP(hipEventCreate(&c->ev_a));
    MGFR_HIP(hipEventCreate(&c->ev_b));
    MGFR_HIP(hipEventCreate(&c->ev_c));
    if (p->precision == MGFR_MIXED) {
        int rc = mixed_alloc(c);
        if (rc) return rc;
    }
    return MGFR_OK;
}

extern "C" int mgfr_create(const mgfr_params *p, void *stream, mgfr_ctx **out)
{
    if (!out) return set_error(MGFR_ERR_ARG, "out is NULL");
    *out = nullptr;
    int rc = validate(p);
    if (rc) return rc;
    mgfr_ctx *c = new (std::nothrow) mgfr_ctx();
    if (!c) return set_error(MGFR_ERR_OOM, "host allocation failed");
    rc = create_impl(p, stream, c);
    if (rc) {
        free_ctx(c);
        return rc;
    }
    *out = c;
    return MGFR_OK;
}

extern "C" void mgfr_destroy(mgfr_ctx *c) { free_ctx(c); }

extern "C" int mgfr_set_stream(mgfr_ctx *c, void *stream)
{
    if (!c) return set_error(MGFR_ERR_ARG, "ctx is NULL");
    c->stream = (hipStream_t)stream;
    return MGFR_OK;
}

extern "C" int mgfr_set_scale_factor(mgfr_ctx *c, double a)
{
    if (!c) return set_error(MGFR_ERR_ARG, "ctx is NULL");
    if (!(a > 0) || !std::isfinite(a)) return set_error(MGFR_ERR_ARG, "a must be > 0 and finite");
    mgfr_params q = c->p;
    q.a = a;
    double fb, beta, C;
    if (int rc = mgfr_background(&q, &fb, &beta, &C)) return rc;
    c->p.a = a;
    c->fbar = fb;
    c->beta = beta;
    c->C = C;
    c->bC = beta * C;
    return MGFR_OK;
}

extern "C" int mgfr_set_timing(mgfr_ctx *c, int on)
{
    if (!c) return set_error(MGFR_ERR_ARG, "ctx is NULL");
    c->timing = on != 0;
    return MGFR_OK;
}

static int check_ptr(const void *p, const char *name)
{
    if (!p) return set_error(MGFR_ERR_ARG, "%s is NULL", name);
    return MGFR_OK;
}

// Form f on level 0 and return D = max|f| (bC if f == 0) on the host.
static int prepare_source(mgfr_ctx *c, const double *delta, double *D)
{
    Level &L0 = c->lev[0];
    size_t n = (size_t)L0.N * L0.N * L0.N;
    double s = c->beta * c->p.omega_m / (c->p.a * c->p.a * c->p.a);
    unsigned g = (unsigned)std::min<size_t>(nblocks(n), (size_t)c->nparts);
    k_source<<<g, kBlock, 0, c->stream>>>(delta, s, n, L0.f, c->partial, (int)g);
    k_final_reduce<<<1, 1024, 0, c->stream>>>(c->partial, (int)g, c->dscal + 2);
    MGFR_HIP(hipGetLastError());
    MGFR_HIP(hipMemcpyAsync(c->hscal + 2, c->dscal + 2, sizeof(double), hipMemcpyDeviceToHost, c->stream));
    MGFR_HIP(hipStreamSynchronize(c->stream));
    double d = c->hscal[2];
    if (!std::isfinite(d)) return set_error(MGFR_ERR_NONFINITE, "delta contains NaN or Inf");
    *D = d > 0 ? d : c->bC;
    return MGFR_OK;
}

// After out-of-place sweeps the current level-0 iterate may sit in the
// context's buffer: copy it back into the caller's array.
static int restore_level0(mgfr_ctx *c, double *user_u)
{
    Level &L0 = c->lev[0];
    if (L0.u != user_u) {
        size_t n = (size_t)L0.N * L0.N * L0.N;
        MGFR_HIP(hipMemcpyAsync(user_u, L0.u, n * sizeof(double), hipMemcpyDeviceToDevice, c->stream));
        L0.alt = L0.u;
        L0.u = user_u;
    }
    return MGFR_OK;
}

static int finish(mgfr_ctx *c, double *u, double *dfr, mgfr_stats *st, int status)
{
    if (dfr) {
        size_t n = (size_t)c->lev[0].N * c->lev[0].N * c->lev[0].N;
        unsigned g = (unsigned)std::min<size_t>(nblocks(n), 8192);
        k_dfr<<<g, kBlock, 0, c->stream>>>(u, c->fbar, n, dfr);
        MGFR_HIP(hipGetLastError());
    }
    MGFR_HIP(hipEventRecord(c->ev_b, c->stream));
    MGFR_HIP(hipEventSynchronize(c->ev_b));
    float ms = 0;
    MGFR_HIP(hipEventElapsedTime(&ms, c->ev_a, c->ev_b));
    if (st) {
        st->t_solve_ms = ms;
        st->status = status;
    }
    if (status == MGFR_ERR_NONFINITE) return set_error(status, "the iteration produced NaN or Inf");
    return status;
}

void mgfr::adapt_smoothing(mgfr_ctx *c, double res, double res2)
{
    if (c->smooth_max <= 0 || !(res2 >= 0.0) || !(res >= res2)) return;
    c->p.pre_smooth = std::min(std::max(1, 2 * c->p.pre_smooth), c->smooth_max);
    c->p.post_smooth = std::min(std::max(1, 2 * c->p.post_smooth), c->smooth_max);
}

// V-cycles on the level-0 iterate, which an odd number of out-of-place sweeps
// leaves in the other buffer: the residual is that of L0.u after every cycle.
int mgfr::solve_fp64_from(mgfr_ctx *c, mgfr_stats *st, double D)
{
    Level &L0 = c->lev[0];
    double rmax, rsq;
    const double ncell = (double)L0.N * L0.N * L0.N;
    int rc = launch_residual_norm64(c, 0, L0.u, L0.f, &rmax, &rsq);
    if (rc) return rc;
    double res = rmax / D, res1 = res, res2 = -1.0;  // res1, res2: one and two checks back
    st->res0 = res;
    int cyc = 0, status;
    for (;;) {
        if (!std::isfinite(res)) { status = MGFR_ERR_NONFINITE; break; }
        if (res <= c->p.tol) { status = MGFR_OK; break; }
        if (cyc >= c->p.max_vcycles) { status = MGFR_NOT_CONVERGED; break; }
        if ((rc = vcycle64(c, 0))) return rc;
        if ((rc = launch_residual_norm64(c, 0, L0.u, L0.f, &rmax, &rsq))) return rc;
        if (c->timing && (rc = collect_timing(c, st))) return rc;
        res2 = cyc >= 1 ? res1 : -1.0;
        res1 = res;
        res = rmax / D;
        adapt_smoothing(c, res, res2);
        if (cyc < MGFR_MAX_HIST) st->res_hist[cyc] = res;
        ++cyc;
    }
    st->vcycles = cyc;
    st->outer_iters = cyc;
    st->res = res;
    st->l2res = std::sqrt(rsq / ncell) / D;
    return status;
}

extern "C" int mgfr_screened_guess(mgfr_ctx *c, const double *delta, double *u)
{
    int rc;
    if ((rc = check_ptr(c, "ctx")) || (rc = check_ptr(delta, "delta")) || (rc = check_ptr(u, "u"))) return rc;
    const size_t n = (size_t)c->lev[0].N * c->lev[0].N * c->lev[0].N;
    const double s = c->p.omega_m / (c->p.a * c->p.a * c->p.a) / c->C;
    const unsigned g = (unsigned)std::min<size_t>((n + kBlock - 1) / kBlock, 16384);
    k_screened_guess<<<g, kBlock, 0, c->stream>>>(delta, s, (double)(c->p.n + 1), n, u);
    MGFR_HIP(hipGetLastError());
    return MGFR_OK;
}

extern "C" int mgfr_effective_density(mgfr_ctx *c, const double *delta, const double *u, double *out)
{
    int rc;
    if ((rc = check_ptr(c, "ctx")) || (rc = check_ptr(delta, "delta")) || (rc = check_ptr(u, "u")) ||
        (rc = check_ptr(out, "out")))
        return rc;
    const size_t n = (size_t)c->lev[0].N * c->lev[0].N * c->lev[0].N;
    const double om = c->p.omega_m / (c->p.a * c->p.a * c->p.a);
    const unsigned g = (unsigned)std::min<size_t>((n + kBlock - 1) / kBlock, 16384);
    k_effective_density<<<g, kBlock, 0, c->stream>>>(delta, u, c->C / (3.0 * om), c->q, n, out);
    MGFR_HIP(hipGetLastError());
    return MGFR_OK;
}

extern "C" int mgfr_solve(mgfr_ctx *c, const double *delta, double *u, double *dfr, mgfr_stats *st_out)
{
    int rc;
    if ((rc = check_ptr(c, "ctx")) || (rc = check_ptr(delta, "delta")) || (rc = check_ptr(u, "u"))) return rc;
    mgfr_stats local;
    mgfr_stats *st = st_out ? st_out : &local;
    memset(st, 0, sizeof *st);
    c->lev[0].u = u;
    c->lev[0].alt = c->alt0;
    c->sweep_timer.used = 0;
    MGFR_HIP(hipEventRecord(c->ev_a, c->stream));
    double D;
    if ((rc = prepare_source(c, delta, &D))) {
        st->status = rc;
        return rc;
    }
    st->scale = D;
    if (c->p.nn_mode == MGFR_NN_COARSE) {
        double tnn = 0;
        if ((rc = nn_warm_start(c, delta, u, &tnn))) return rc;
        st->t_nn_ms = tnn;
    }
    int status;
    const int pre = c->p.pre_smooth, post = c->p.post_smooth;  // adaptive smoothing changes them per solve
    if (c->p.precision == MGFR_MIXED) {
        status = solve_mixed(c, u, st, D);
    } else {
        status = solve_fp64_from(c, st, D);
    }
    st->smooth_used = c->p.pre_smooth;
    c->p.pre_smooth = pre;
    c->p.post_smooth = post;
    if (status < 0 && status != MGFR_ERR_NONFINITE) return status;
    if ((rc = restore_level0(c, u))) return rc;
    return finish(c, u, dfr, st, status);
}

extern "C" int mgfr_ngs_sweep(mgfr_ctx *c, double *u, const double *f, int sweeps)
{
    int rc;
    if ((rc = check_ptr(c, "ctx")) || (rc = check_ptr(u, "u")) || (rc = check_ptr(f, "f"))) return rc;
    if (sweeps < 0) return set_error(MGFR_ERR_ARG, "sweeps must be >= 0");
    Level &L0 = c->lev[0];
    L0.u = u;
    L0.alt = c->alt0;
    if ((rc = launch_sweep64(c, 0, nullptr, f, sweeps, false))) return rc;
    if ((rc = restore_level0(c, u))) return rc;
    MGFR_HIP(hipStreamSynchronize(c->stream));
    return MGFR_OK;
}

extern "C" int mgfr_set_fused_min_mesh(mgfr_ctx *c, int n)
{
    if (!c) return set_error(MGFR_ERR_ARG, "ctx is NULL");
    if (n != 0 && n < 64) return set_error(MGFR_ERR_ARG, "fused sweeps need levels of at least 64^3 (or 0 = off)");
    c->fused_min_n = n;
    return MGFR_OK;
}

extern "C" int mgfr_set_colour_min_mesh(mgfr_ctx *c, int n)
{
    if (!c) return set_error(MGFR_ERR_ARG, "ctx is NULL");
    if (n != 0 && n < 128) return set_error(MGFR_ERR_ARG, "one-colour pass kernels need levels of at least 128^3 (or 0 = off)");
    c->colour32_min_n = n;
    return MGFR_OK;
}

extern "C" int mgfr_set_relaxation32(mgfr_ctx *c, double omega)
{
    if (!c) return set_error(MGFR_ERR_ARG, "ctx is NULL");
    if (!(omega > 0.0 && omega < 2.0)) return set_error(MGFR_ERR_ARG, "omega must be in (0, 2)");
    c->omega32 = omega;
    return MGFR_OK;
}

extern "C" int mgfr_set_adaptive_smoothing(mgfr_ctx *c, int max_sweeps)
{
    if (!c) return set_error(MGFR_ERR_ARG, "ctx is NULL");
    if (max_sweeps != 0 && (max_sweeps < std::max(c->p.pre_smooth, c->p.post_smooth) || max_sweeps > 32))
        return set_error(MGFR_ERR_ARG, "max_sweeps must be 0 or in [max(pre_smooth, post_smooth), 32]");
    c->smooth_max = max_sweeps;
    return MGFR_OK;
}

extern "C" int mgfr_set_inner_cycles(mgfr_ctx *c, int max_inner)
{
    if (!c) return set_error(MGFR_ERR_ARG, "ctx is NULL");
    if (max_inner < 1 || max_inner > 4) return set_error(MGFR_ERR_ARG, "max_inner must be in [1, 4]");
    c->inner_max = max_inner;
    return MGFR_OK;
}

extern "C" int mgfr_set_fused_sweep32(mgfr_ctx *c, int on)
{
    if (!c) return set_error(MGFR_ERR_ARG, "ctx is NULL");
    if (on != 0 && on != 1) return set_error(MGFR_ERR_ARG, "on must be 0 or 1");
    if (on && c->p.precision == MGFR_MIXED && c->lev[0].N >= 128 && !c->lev[0].e32alt)
        return set_error(MGFR_ERR_ARG, "no second correction buffer (the context was not created for mixed precision)");
    c->fused32 = on;
    return MGFR_OK;
}

extern "C" int mgfr_vcycle(mgfr_ctx *c, double *u, const double *f)
{
    int rc;
    if ((rc = check_ptr(c, "ctx")) || (rc = check_ptr(u, "u")) || (rc = check_ptr(f, "f"))) return rc;
    Level &L0 = c->lev[0];
    size_t n = (size_t)L0.N * L0.N * L0.N;
    MGFR_HIP(hipMemcpyAsync(L0.f, f, n * sizeof(double), hipMemcpyDeviceToDevice, c->stream));
    L0.u = u;
    L0.alt = c->alt0;
    if ((rc = vcycle64(c, 0))) return rc;
    if ((rc = restore_level0(c, u))) return rc;
    MGFR_HIP(hipStreamSynchronize(c->stream));
    return MGFR_OK;
}

extern "C" int mgfr_residual(mgfr_ctx *c, const double *u, const double *f, double *r)
{
    int rc;
    if ((rc = check_ptr(c, "ctx")) || (rc = check_ptr(u, "u")) || (rc = check_ptr(f, "f")) ||
        (rc = check_ptr(r, "r")))
        return rc;
    Level &L0 = c->lev[0];
    size_t n = (size_t)L0.N * L0.N * L0.N;
    k_residual_field<<<nblocks(n), kBlock, 0, c->stream>>>(u, f, L0.lg, level_const(c, 0), r);
    MGFR_HIP(hipGetLastError());
    MGFR_HIP(hipStreamSynchronize(c->stream));
    return MGFR_OK;
}
