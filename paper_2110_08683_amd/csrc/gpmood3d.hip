// 3D GP-MOOD stage (GP-MOOD5 and lower) for gfx950, with its C ABI (gpm3_*).
//
// The 3D form of the method (3D is future work in the paper; readings as in the
// 3D oracle): five conservative variables (rho, rho u, rho v, rho w, E), the GP
// stencil of radius R <= 2 is the L1 ball (7 / 25 cells), a face carries the q x q
// tensor Gauss nodes (q = R + 1), EDP_1 face orders, HLLC with two tangential
// momenta, detection with the six face neighbours (DMP, plateau, CSD with the z
// terms, u2 per direction), SSP-RK3 (eq. (rk3)), FP64 CFL dt.
//
// Kernels:
//   k3_faces_line, k3_faces_march  the first evaluation at radius 2: every face, a cell's
//             ball read once for its two faces on the axis (k3_faces_top: radius 1, one
//             thread per face).
//   k3_faces  the claimed faces of a cascade pass, one thread per face: both cells' node
//             states at the face's EDP_1 radius (dot products with the quad-precision
//             weights), q^2 HLLC solves, the Gauss sum; flux and Riemann-state flags
//             stored.
//   k3_cells  one thread per cell: candidate from the six stored fluxes,
//             detection, RK combination, lowering and claims (stamps, one atomic
//             per wavefront and list) of the faces and cells of the next pass.
// The MOOD loop is the synchronous iteration of the 2D engine: a pass recomputes
// the claimed faces, then re-evaluates the claimed cells, until no cell is
// troubled.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "gp_weights.h"
#include "gpmood.h"
#include "gpmood_device.h"

namespace gpm {

constexpr int kZ3 = 6 * 9 * 25;  // weights per radius: [6 faces][9 nodes][25 cells]
constexpr int kPZ3 = 6 * 4 * kNPar3;  // radius-2 parity weights: [6 faces][4 node classes][25 entries]

template <typename real>
struct Stage3 {
    const real *Un;
    const real *Us;
    real *Uout;
    const double *dt;
    uint8_t *order;
    real *F[3];          // per axis a: [5][nz + (a == 2)][ny + (a == 1)][nx + (a == 0)]
    uint8_t *Ff[3];      // bit 0 / 1: the left / right state is inadmissible
    unsigned *cstamp;    // [ncell]
    unsigned *fstamp;    // [all faces, axes concatenated]
    int n[3], bc[3];
    int fofs[4];         // first face id of each axis, total
    int s, top;
    unsigned flags;
    int next[4];
    real d[3], gamma, sigma_v, sigma_p, plat_thr, delta;
    const real *z;       // [R - 1][6][9][25]
    const real *qw;      // [R - 1][9]
    const real *pz;      // [6][4][25]: radius 2 in the parity basis (kPar3)
    real curv[3][4];
    const unsigned *stamp0;
};

typedef const __attribute__((address_space(1))) char *global_bytes;

// Index of (a, b), |a| + |b| <= 2, among the 13 offsets of the ball off one axis.
__host__ __device__ constexpr int disc_index(int a, int b)
{
    return a == -2 ? 0 : (a == -1 ? 2 + b : (a == 0 ? 6 + b : (a == 1 ? 10 + b : 12)));
}

struct PassOut3 {
    int *flist, *fcount, *clist, *ccount, *tcount;
    unsigned stamp;
};

__device__ __forceinline__ int w3(int i, int n, int bc)
{
    if (bc == 0) return i < 0 ? i + n : (i >= n ? i - n : i);
    return i < 0 ? 0 : (i >= n ? n - 1 : i);
}

template <typename real>
__device__ __forceinline__ size_t cell3(const Stage3<real> &S, int i, int j, int k)
{
    return ((size_t)w3(k, S.n[2], S.bc[2]) * S.n[1] + w3(j, S.n[1], S.bc[1])) * S.n[0] + w3(i, S.n[0], S.bc[0]);
}

template <typename real>
__device__ __forceinline__ real p3(real g, const real (&q)[5])
{
    return (g - real(1)) * (q[4] - dv(real(0.5) * (q[1] * q[1] + q[2] * q[2] + q[3] * q[3]), q[0]));
}

// HLLC with normal axis a (1 + a is the normal momentum), as the 2D solver with a
// second tangential momentum.
template <typename real>
__device__ __forceinline__ void hllc3(real g, int a, const real (&UL)[5], const real (&UR)[5], real (&F)[5],
                                      bool &badL, bool &badR)
{
    const int n = 1 + a, t1 = 1 + (a + 1) % 3, t2 = 1 + (a + 2) % 3;
    const real rl = UL[0], irl = dv(real(1), rl), ul = UL[n] * irl, vl = UL[t1] * irl, wl = UL[t2] * irl, El = UL[4];
    const real rr = UR[0], irr = dv(real(1), rr), ur = UR[n] * irr, vr = UR[t1] * irr, wr = UR[t2] * irr, Er = UR[4];
    const real pl = (g - real(1)) * (El - real(0.5) * rl * (ul * ul + vl * vl + wl * wl));
    const real pr = (g - real(1)) * (Er - real(0.5) * rr * (ur * ur + vr * vr + wr * wr));
    badL = !(pos_finite(rl) && pos_finite(pl));
    badR = !(pos_finite(rr) && pos_finite(pr));
    const real cl = sq(g * pl * irl), cr = sq(g * pr * irr);
    const real SL = vmin(ul - cl, ur - cr);
    const real SR = vmax(ul + cl, ur + cr);
    const real Ss = dv(pr - pl + rl * ul * (SL - ul) - rr * ur * (SR - ur), rl * (SL - ul) - rr * (SR - ur));
    const bool useL = Ss >= real(0);
    const bool takeL = SL >= real(0);
    const bool takeStar = !takeL && (useL || SR > real(0));
    // the side whose state the flux needs, in every branch (as in 2D)
    const bool left = takeL || useL;
    const real rk = left ? rl : rr, uk = left ? ul : ur, vk = left ? vl : vr, wk = left ? wl : wr;
    const real Ek = left ? El : Er, pk = left ? pl : pr, Sk = left ? SL : SR, irk = left ? irl : irr;
    const real sku = Sk - uk;
    const real fac = dv(rk * sku, Sk - Ss);
    const real fk[5] = {rk * uk, rk * uk * uk + pk, rk * uk * vk, rk * uk * wk, uk * (Ek + pk)};
    const real uc[5] = {rk, rk * uk, rk * vk, rk * wk, Ek};
    const real us[5] = {fac, fac * Ss, fac * vk, fac * wk, fac * (Ek * irk + (Ss - uk) * (Ss + dv(pk, rk * sku)))};
    real f[5];
#pragma unroll
    for (int m = 0; m < 5; ++m) {
        const real fs = fk[m] + Sk * (us[m] - uc[m]);
        f[m] = takeStar ? fs : fk[m];
    }
    F[0] = f[0];
    F[4] = f[4];
#pragma unroll
    for (int m = 1; m < 4; ++m) F[m] = m == n ? f[1] : (m == t1 ? f[2] : f[3]);
}

// Decode a face id: axis a, and the cell (i, j, k) on its + side (the left cell is
// one step back along a).
template <typename real>
__device__ __forceinline__ void face3_decode(const Stage3<real> &S, int f, int &a, int &i, int &j, int &k, int &loc)
{
    a = f < S.fofs[1] ? 0 : (f < S.fofs[2] ? 1 : 2);
    loc = f - S.fofs[a];
    const int m0 = S.n[0] + (a == 0), m1 = S.n[1] + (a == 1);
    i = loc % m0;
    const int r = loc / m0;
    j = r % m1;
    k = r / m1;
}

template <typename real>
__device__ __forceinline__ void face3_flux(const Stage3<real> &S, int f)
{
    int a, i, j, k, loc;
    face3_decode(S, f, a, i, j, k, loc);
    const int iL = i - (a == 0), jL = j - (a == 1), kL = k - (a == 2);
    const int R = min((int)S.order[cell3(S, iL, jL, kL)], (int)S.order[cell3(S, i, j, k)]);
    const size_t plane = (size_t)S.n[0] * S.n[1] * S.n[2];
    real Fs[5] = {real(0), real(0), real(0), real(0), real(0)};
    bool bl = false, br = false;
    if (R <= 0) {
        real UL[5], UR[5];
        const size_t cl = cell3(S, iL, jL, kL), cr = cell3(S, i, j, k);
#pragma unroll
        for (int v = 0; v < 5; ++v) {
            UL[v] = S.Us[v * plane + cl];
            UR[v] = S.Us[v * plane + cr];
        }
        real fl[5];
        hllc3(S.gamma, a, UL, UR, fl, bl, br);
#pragma unroll
        for (int v = 0; v < 5; ++v) Fs[v] = fma(real(1), fl[v], real(0));
    } else {
        const int ns = R == 1 ? 7 : 25, nq = R == 1 ? 4 : 9;
        const real *zL = S.z + ((size_t)(R - 1) * 6 + 2 * a + 1) * 9 * 25;  // + face of the left cell
        const real *zR = S.z + ((size_t)(R - 1) * 6 + 2 * a) * 9 * 25;      // - face of the right cell
        real st[9][2][5];
#pragma unroll
        for (int v = 0; v < 5; ++v) {
            real qL[25], qR[25];
#pragma unroll
            for (int m = 0; m < 25; ++m) {
                if (m < ns) {
                    qL[m] = S.Us[v * plane + cell3(S, iL + kBall[m][0], jL + kBall[m][1], kL + kBall[m][2])];
                    qR[m] = S.Us[v * plane + cell3(S, i + kBall[m][0], j + kBall[m][1], k + kBall[m][2])];
                } else {
                    qL[m] = qR[m] = real(0);
                }
            }
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                real sl = real(0), sr = real(0);
                if (q < nq) {
#pragma unroll
                    for (int m = 0; m < 25; ++m)
                        if (m < ns) {
                            sl = fma(zL[q * 25 + m], qL[m], sl);
                            sr = fma(zR[q * 25 + m], qR[m], sr);
                        }
                }
                st[q][0][v] = sl;
                st[q][1][v] = sr;
            }
        }
        const real *w = S.qw + (size_t)(R - 1) * 9;
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            if (q < nq) {
                real fl[5];
                bool b1, b2;
                hllc3(S.gamma, a, st[q][0], st[q][1], fl, b1, b2);
                bl = bl || b1;
                br = br || b2;
#pragma unroll
                for (int v = 0; v < 5; ++v) Fs[v] = fma(w[q], fl[v], Fs[v]);
            }
        }
    }
    const int m0 = S.n[0] + (a == 0), m1 = S.n[1] + (a == 1), m2 = S.n[2] + (a == 2);
    const size_t nfa = (size_t)m0 * m1 * m2;
#pragma unroll
    for (int v = 0; v < 5; ++v) S.F[a][v * nfa + loc] = Fs[v];
    S.Ff[a][loc] = (uint8_t)((bl ? 1 : 0) | (br ? 2 : 0));
}

template <typename real>
__global__ __launch_bounds__(128) void k3_faces(const Stage3<real> S, const int *list, const int *count)
{
    const int cap = S.fofs[3];
    int n = *count;
    n = n < cap ? n : cap;
    for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x) face3_flux(S, list[t]);
}

// First evaluation at top radius 1: every face of axis A (every cell starts the
// stage at the top order), with the products and sums of face3_flux in the same
// order.  All 2 x 5 stencils are loaded once into registers; the node loop is
// rolled and reads each node's 2 x 7 weights through the scalar path (A is
// uniform), so no lane loads a weight.
template <typename real, int A>
__global__ __launch_bounds__(128, 1) void k3_faces_top(const Stage3<real> S)
{
    constexpr int ns = 7, nq = 4;
    const int m0 = S.n[0] + (A == 0), m1 = S.n[1] + (A == 1), m2 = S.n[2] + (A == 2);
    const int nfa = m0 * m1 * m2;
    const int loc = blockIdx.x * blockDim.x + threadIdx.x;
    if (loc >= nfa) return;
    const size_t plane = (size_t)S.n[0] * S.n[1] * S.n[2];
    const int i = loc % m0, rr = loc / m0, j = rr % m1, k = rr / m1;
    const int iL = i - (A == 0), jL = j - (A == 1), kL = k - (A == 2);
    real qL[5][ns], qR[5][ns];
#pragma unroll
    for (int m = 0; m < ns; ++m) {
        const size_t cl = cell3(S, iL + kBall[m][0], jL + kBall[m][1], kL + kBall[m][2]);
        const size_t cr = cell3(S, i + kBall[m][0], j + kBall[m][1], k + kBall[m][2]);
#pragma unroll
        for (int v = 0; v < 5; ++v) {
            qL[v][m] = S.Us[v * plane + cl];
            qR[v][m] = S.Us[v * plane + cr];
        }
    }
    const cptr<real> zL = (cptr<real>)S.z + (2 * A + 1) * 9 * 25;  // + face of the left cell
    const cptr<real> zR = (cptr<real>)S.z + 2 * A * 9 * 25;        // - face of the right cell
    const cptr<real> w = (cptr<real>)S.qw;
    real Fs[5] = {real(0), real(0), real(0), real(0), real(0)};
    bool bl = false, br = false;
#pragma unroll 1
    for (int q = 0; q < nq; ++q) {
        real sl[5], sr[5];
#pragma unroll
        for (int v = 0; v < 5; ++v) {
            real a = real(0), b = real(0);
#pragma unroll
            for (int m = 0; m < ns; ++m) {
                a = fma(zL[q * 25 + m], qL[v][m], a);
                b = fma(zR[q * 25 + m], qR[v][m], b);
            }
            sl[v] = a;
            sr[v] = b;
        }
        real fl[5];
        bool b1, b2;
        hllc3(S.gamma, A, sl, sr, fl, b1, b2);
        bl = bl || b1;
        br = br || b2;
#pragma unroll
        for (int v = 0; v < 5; ++v) Fs[v] = fma(w[q], fl[v], Fs[v]);
    }
#pragma unroll
    for (int v = 0; v < 5; ++v) S.F[A][(size_t)v * nfa + loc] = Fs[v];
    S.Ff[A][loc] = (uint8_t)((bl ? 1 : 0) | (br ? 2 : 0));
}

// Radius 2 in the parity basis: per variable, a cell's 25
// ball values are folded into the 25 parity entries of the face axis (kPar3) and
// the nine node states come from the four node classes' weights: 14 products for
// the centre, 19 for each pair on a tangential axis, 25 for the four corners (77,
// against 225 for nine 25-term dot products).  The weights are the orbit
// averages of the quad-precision prediction vectors; the node states agree with
// the plain dot products to rounding.
template <int A>
__device__ __forceinline__ constexpr int par_member(int e, int s1, int s2)
{
    const int t1 = A == 0 ? 1 : 0, t2 = A == 2 ? 1 : 2;
    int d[3] = {0, 0, 0};
    d[A] = kPar3[e].dn;
    d[t1] = s1 * kPar3[e].a1;
    d[t2] = s2 * kPar3[e].a2;
    return ball_index(d[0], d[1], d[2]);
}

template <int A, typename real>
__device__ __forceinline__ void par3_entries(const real (&q)[25], real (&P)[kNPar3])
{
#pragma unroll
    for (int e = 0; e < kNPar3; ++e) {
        const int a1 = kPar3[e].a1, a2 = kPar3[e].a2, c = kPar3[e].comp;
        const real pp = q[par_member<A>(e, 1, 1)];
        if (a1 == 0 && a2 == 0) {
            P[e] = pp;
        } else if (a2 == 0) {
            const real mp = q[par_member<A>(e, -1, 1)];
            P[e] = c == 0 ? pp + mp : pp - mp;
        } else if (a1 == 0) {
            const real pm = q[par_member<A>(e, 1, -1)];
            P[e] = c == 0 ? pp + pm : pp - pm;
        } else {
            const real mp = q[par_member<A>(e, -1, 1)], pm = q[par_member<A>(e, 1, -1)];
            const real mm = q[par_member<A>(e, -1, -1)];
            P[e] = c == 0 ? (pp + mp) + (pm + mm)
                 : c == 1 ? (pp - mp) + (pm - mm)
                 : c == 2 ? (pp + mp) - (pm + mm)
                          : (pp - mp) - (pm - mm);
        }
    }
}

// Sum of the entries E0..E1-1 with weights w[0..]; the products in order of the entry.
template <int E0, int E1, typename real>
__device__ __forceinline__ real par3_dot(const real *w, const real (&P)[kNPar3])
{
    real s = real(0);
#pragma unroll
    for (int e = E0; e < E1; ++e) s = fma(w[e], P[e], s);
    return s;
}

// The nine node states (table order) of one face side from its parity entries.  The
// 77 weights are read through the scalar path, all at once in FP32 and in two lots in
// FP64 (66 and 88 scalar registers), and given up before the next are read.
template <typename real>
__device__ __forceinline__ void par3_states(const real (&P)[kNPar3], cptr<real> W, real (&s)[9])
{
    constexpr int EE = kPar3EE, OE = EE + kPar3OE, EO = OE + kPar3EO;
    real w[4][kNPar3];
    auto load = [&](int cls) {
        const cptr<real> Wc = W;
#pragma unroll
        for (int e = 0; e < kNPar3; ++e) w[cls][e] = Wc[cls * kNPar3 + e];
    };
    W = reread(W);
    load(0);
    load(1);
    if constexpr (sizeof(real) == 4) {
        load(2);
        load(3);
        __builtin_amdgcn_sched_barrier(0);
    }
    real x[4];
    x[0] = par3_dot<0, EE>(w[0], P);
    x[1] = par3_dot<0, EE>(w[1], P);
    x[2] = par3_dot<EE, OE>(w[1], P);
    x[3] = real(0);
    if constexpr (sizeof(real) == 8) {
        hold(x);
        __builtin_amdgcn_sched_barrier(0);
        W = reread(W);
        load(2);
        load(3);
    }
    s[4] = x[0];
    s[1] = x[1] + x[2];
    s[7] = x[1] - x[2];
    const real a2 = par3_dot<0, EE>(w[2], P), c2 = par3_dot<OE, EO>(w[2], P);
    s[3] = a2 + c2;
    s[5] = a2 - c2;
    const real a3 = par3_dot<0, EE>(w[3], P), b3 = par3_dot<EE, OE>(w[3], P), c3 = par3_dot<OE, EO>(w[3], P);
    const real d3 = w[3][kNPar3 - 1] * P[kNPar3 - 1];
    s[0] = (a3 + b3) + (c3 + d3);
    s[2] = (a3 + b3) - (c3 + d3);
    s[6] = (a3 - b3) + (c3 - d3);
    s[8] = (a3 - b3) - (c3 - d3);
    hold(s);
    __builtin_amdgcn_sched_barrier(0);
}

// The lane's byte offsets into a variable are 32-bit (OFF), so that a load takes a scalar
// base and one register: held in place by hold(), widened outside a loop they cost an add
// and a register each.
template <typename real, typename OFF, int N, typename Sel, typename Base>
__device__ __forceinline__ void ball3(OFF (&off)[N], real (&q)[25], Base base, Sel sel)
{
    hold(off);
#pragma unroll
    for (int m = 0; m < 25; ++m)
        q[m] = *(const __attribute__((address_space(1))) real *)(base(m) + off[sel(m)]);
}

// The nine HLLC solves of a face and their Gauss sum; left(n, sl) gives node n's left state.
template <int A, typename real, typename Left>
__device__ __forceinline__ void gauss3(const Stage3<real> &K, const real (&sm)[9][5], Left left, real (&Fs)[5], int &bad)
{
    const cptr<real> w = (cptr<real>)K.qw + 9;
    bool bl = false, br = false;
#pragma unroll
    for (int v = 0; v < 5; ++v) Fs[v] = real(0);
#pragma unroll
    for (int n = 0; n < 9; ++n) {
        real sl[5], fl[5];
        left(n, sl);
        bool b1, b2;
        hllc3(K.gamma, A, sl, sm[n], fl, b1, b2);
        bl = bl || b1;
        br = br || b2;
#pragma unroll
        for (int v = 0; v < 5; ++v) Fs[v] = fma(w[n], fl[v], Fs[v]);
        hold(Fs);
        __builtin_amdgcn_sched_barrier(0);
    }
    bad = (bl ? 1 : 0) | (br ? 2 : 0);
}

// One variable's states of a cell on its - face (sm) and + face (sp) of axis A.
template <int A, typename real>
__device__ __forceinline__ void sides3(const Stage3<real> &S, const real (&P)[kNPar3], int v, real (&sm)[9][5],
                                       real (&sp)[9][5])
{
    const cptr<real> W = (cptr<real>)S.pz + 2 * A * 4 * kNPar3;
    real st[9];
    par3_states(P, W, st);
#pragma unroll
    for (int n = 0; n < 9; ++n) sm[n][v] = st[n];
    par3_states(P, W + 4 * kNPar3, st);
#pragma unroll
    for (int n = 0; n < 9; ++n) sp[n][v] = st[n];
}

// First evaluation at radius 2 (k3_faces_line, k3_faces_march): a cell's ball is read once
// for both of its faces on the axis, whose states share the parity entries, and a face
// takes its left state from the cell one step back.  Bound by vector instructions (about
// 2300 a cell in FP32) and, at three or four wavefronts a SIMD, the waits between them.
// One thread per face that read both balls, with two wavefronts a SIMD in FP32 and one in
// FP64, took 784, 780 and 705 us on x, y and z at 192^3 in FP32 and 163, 161 and 151 us at
// 97 x 64 x 81 in FP64; now 337, 429 and 422 us, and 76, 108 and 107 us.  A tile of eight lanes
// along y or z by eight columns, which needs no march, took 1000 us: a load of eight short
// rows takes the cache twice as long as one of 64 cells in a row.
//
// k3_faces_line: the cell one step back is the lane `step` below (1 on x, n_x on y, n_x n_y
// on z): a wavefront runs 64 positions of the lines written one after the other, a ghost cell
// at either end of each included, and writes 64 - step faces.
template <typename real, int A, typename OFF>
__global__ __launch_bounds__(64, sizeof(real) == 4 ? 4 : 2) void k3_faces_line(const Stage3<real>)
{
    const Stage3<real> &S = first_arg<Stage3<real>>();
    const int step = A == 0 ? 1 : (A == 1 ? S.n[0] : S.n[0] * S.n[1]);
    int pos[3], loc;
    bool live;
    {
        const int len = step * (S.n[A] + 2), lane = threadIdx.x;
        const int total = len * (A == 0 ? S.n[1] * S.n[2] : (A == 1 ? S.n[2] : 1));
        const int q = (64 - step) * xcd_tile(blockIdx.x, gridDim.x) + lane, qc = min(q, total - 1), r = qc / len;
        const int o = qc - r * len, h = o / step, in = o - h * step;
        if constexpr (A == 0) {
            pos[1] = r % S.n[1];
            pos[2] = r / S.n[1];
        } else if constexpr (A == 1) {
            pos[0] = in;
            pos[2] = r;
        } else {
            pos[0] = in % S.n[0];
            pos[1] = in / S.n[0];
        }
        pos[A] = h - 1;  // -1 and n: the ghost cells
        live = lane >= step && pos[A] >= 0 && q < total;
        loc = (r * (S.n[A] + 1) + pos[A]) * step + in;
    }
    OFF off[25];
    {
        const OFF row = (OFF)S.n[0] * (OFF)sizeof(real), stride[3] = {(OFF)sizeof(real), row, row * (OFF)S.n[1]};
        OFF o[3][5];
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int d = 0; d < 5; ++d) o[a][d] = (OFF)w3(pos[a] + d - 2, S.n[a], S.bc[a]) * stride[a];
#pragma unroll
        for (int m = 0; m < 25; ++m) off[m] = o[0][kBall[m][0] + 2] + o[1][kBall[m][1] + 2] + o[2][kBall[m][2] + 2];
    }
    auto fetch = [&](int v, real (&q)[25]) {
        const Stage3<real> &K = *(const Stage3<real> *)reread((cptr<Stage3<real>>)&S);
        const global_bytes U = (global_bytes)(K.Us + (size_t)v * K.n[0] * K.n[1] * K.n[2]);
        ball3(off, q, [&](int) { return U; }, [](int m) { return m; });
    };
    real qn[25], sm[9][5], sp[9][5];
    fetch(0, qn);
#pragma unroll
    for (int v = 0; v < 5; ++v) {
        real P[kNPar3];
        par3_entries<A>(qn, P);
        hold(P);
        if (v < 4) fetch(v + 1, qn);  // in flight during this variable's products
        __builtin_amdgcn_sched_barrier(0);
        sides3<A>(S, P, v, sm, sp);
    }
    const Stage3<real> &K = *(const Stage3<real> *)reread((cptr<Stage3<real>>)&S);
    real Fs[5];
    int bad;
    gauss3<A>(
        K, sm,
        [&](int n, real (&sl)[5]) {
#pragma unroll
            for (int v = 0; v < 5; ++v) sl[v] = A == 0 ? lane_shift<-1>(sp[n][v]) : __shfl_up(sp[n][v], step);
        },
        Fs, bad);
    if (!live) return;
    const size_t nfa = (size_t)(K.n[0] + (A == 0)) * (K.n[1] + (A == 1)) * (K.n[2] + (A == 2));
#pragma unroll
    for (int v = 0; v < 5; ++v) K.F[A][v * nfa + loc] = Fs[v];
    K.Ff[A][loc] = (uint8_t)bad;
}

// On y and z a lane marches along the axis over `len` faces, the + states of the cell
// before kept from one step to the next: in LDS, but for the last node's in FP64 (45
// values a lane are 23 KB a wavefront, 40 are an eighth of a CU's LDS, which two
// wavefronts on each SIMD take).  The 64 lanes are consecutive columns, x fastest, and
// every load's offset along the axis is scalar.
template <typename real, int A, typename OFF>
__global__ __launch_bounds__(64, sizeof(real) == 4 ? 3 : 2) void k3_faces_march(const Stage3<real>, int len)
{
    constexpr int t2 = 3 - A;                        // the other axis of the columns
    constexpr int kept = sizeof(real) == 4 ? 45 : 40;  // + states held in LDS
    __shared__ real prev[kept][64];
    const Stage3<real> &S = first_arg<Stage3<real>>();
    const int lane = threadIdx.x;
    int lo, hi, loc;
    bool live;
    OFF off[13];
    {
        const int cols = S.n[0] * S.n[t2], groups = (cols + 63) / 64;
        const int wave = xcd_tile(blockIdx.x, gridDim.x), seg = wave / groups;
        const int col = (wave - seg * groups) * 64 + lane, cc = min(col, cols - 1);
        const int px = cc % S.n[0], pt = cc / S.n[0];
        lo = seg * len;
        hi = min(lo + len, S.n[A] + 1);
        live = col < cols;
        loc = (A == 1 ? pt * (S.n[1] + 1) : pt) * S.n[0] + px;  // face 0 of the column
        const OFF row = (OFF)S.n[0] * (OFF)sizeof(real), stride = A == 1 ? row * (OFF)S.n[1] : row;
        OFF ox[5], ot[5];
#pragma unroll
        for (int d = 0; d < 5; ++d) {
            ox[d] = (OFF)w3(px + d - 2, S.n[0], S.bc[0]) * (OFF)sizeof(real);
            ot[d] = (OFF)w3(pt + d - 2, S.n[t2], S.bc[t2]) * stride;
        }
#pragma unroll
        for (int m = 0; m < 25; ++m) off[disc_index(kBall[m][0], kBall[m][t2])] = ox[kBall[m][0] + 2] + ot[kBall[m][t2] + 2];
    }
    // cell indices of the five positions along the axis about cell c (scalar)
    int r[5];
    auto rows = [&](int c) {
#pragma unroll
        for (int d = 0; d < 5; ++d) {
            const int i = c + d - 2, n = S.n[A];
            const int p = i < 0 ? i + n : (i >= n ? i - n : i), q = min(max(i, 0), n - 1);
            r[d] = S.bc[A] == 0 ? p : q;
        }
    };
    auto fetch = [&](int v, real (&q)[25]) {
        const Stage3<real> &K = *(const Stage3<real> *)reread((cptr<Stage3<real>>)&S);
        const size_t row = sizeof(real) * (size_t)K.n[0], slab = row * K.n[1];
        const global_bytes U = (global_bytes)K.Us + v * slab * K.n[2];
        global_bytes Ur[5];
#pragma unroll
        for (int d = 0; d < 5; ++d) {
            Ur[d] = U + (size_t)r[d] * (A == 1 ? row : slab);
            asm volatile("" : "+s"(Ur[d]));  // stays a scalar base
        }
        ball3(off, q, [&](int m) { return Ur[kBall[m][A] + 2]; },
              [](int m) { return disc_index(kBall[m][0], kBall[m][t2]); });
    };
    real qn[25], last[5];
    auto next = [&](int c) {
        rows(min(c + 1, hi - 1));
        fetch(0, qn);
    };
    rows(lo - 1);
    fetch(0, qn);
#pragma unroll 1
    for (int c = lo - 1; c < hi; ++c) {
        real sm[9][5], sp[9][5];
#pragma unroll
        for (int v = 0; v < 5; ++v) {
            real P[kNPar3];
            par3_entries<A>(qn, P);
            hold(P);
            // the next variable's loads are in flight during this one's products; the next
            // cell's first in FP32 too (in FP64 the registers hold both sides' states then)
            if (v < 4) fetch(v + 1, qn);
            else if (kept == 45) next(c);
            __builtin_amdgcn_sched_barrier(0);
            sides3<A>(S, P, v, sm, sp);
        }
        auto keep = [&](int n) {
#pragma unroll
            for (int v = 0; v < 5; ++v) {
                if (5 * n + v < kept) prev[5 * n + v][lane] = sp[n][v];
                else last[v] = sp[n][v];
            }
        };
        if (c < lo) {
#pragma unroll
            for (int n = 0; n < 9; ++n) keep(n);
            if (kept != 45) next(c);
            continue;
        }
        const Stage3<real> &K = *(const Stage3<real> *)reread((cptr<Stage3<real>>)&S);
        real Fs[5];
        int bad;
        gauss3<A>(
            K, sm,
            [&](int n, real (&sl)[5]) {
#pragma unroll
                for (int v = 0; v < 5; ++v) sl[v] = 5 * n + v < kept ? prev[5 * n + v][lane] : last[v];
                keep(n);
            },
            Fs, bad);
        if (kept != 45) next(c);
        if (!live) continue;
        const int k1 = K.n[1] + (A == 1);
        const size_t nfa = (size_t)K.n[0] * k1 * (K.n[2] + (A == 2));
        const size_t f = (size_t)loc + (size_t)c * (size_t)(A == 1 ? K.n[0] : K.n[0] * K.n[1]);
#pragma unroll
        for (int v = 0; v < 5; ++v) K.F[A][v * nfa + f] = Fs[v];
        K.Ff[A][f] = (uint8_t)bad;
    }
}

// Faces per march of k3_faces_march on axis a: the longest of at most 6 that leaves three
// marches for each of the 1024 SIMDs.  A march of T faces runs T + 1 cells, so a long one
// runs fewer in all; but with fewer marches than that a SIMD waits on memory, and past 6
// faces the last round of marches costs more than the extra cells.  Microseconds a step at
// 1, 2, 3, 4, 6, 8, 12 faces: 32^3 FP64 275 334 377 432 547 666 890; 97 x 64 x 81 FP64
// 1184 1075 1075 1101 1136 1294 1426; 64^3 FP32 418 414 423 473 527 609 731; 192^3 FP32
// 5760 5000 4830 4700 4650 4730 4750, FP64 13510 11730 11300 11050 10850 10930 10940.
static int march3(const int (&n)[3], int a, long long groups)
{
    int T = 6;
    while (T > 1 && groups * ((n[a] + T) / T) < 3 * 1024) --T;
    return T;
}

// On y and z k3_faces_line takes the grids that are thin below the axis: there the march's 64
// columns lie in many short rows, or are fewer than the lanes, while the line still reads one
// run of memory and gives up step of its 64 lanes.  Microseconds a smooth step, line against
// march: FP32 1 x 400 x 400 292 499, 3 x 600 x 600 911 1408, 8 x 350 x 350 799 888,
// 16 x 256 x 256 854 915, 24 x 200 x 200 781 757, 32 x 200 x 200 1122 1058; FP64 549 752,
// 1860 2107, 1659 1743, 1737 1764, 1652 1578, 2365 2111.  With few columns FP32 (FP64)
// 1 x 8 x 4000 174 290 (223 411), 24 x 1 x 4000 259 287 (448 497).
constexpr int kLineStep = 16, kLineCols = 32;

template <typename real, int A, typename OFF>
static void launch_line(const Stage3<real> &S, hipStream_t st)
{
    const int step = A == 0 ? 1 : (A == 1 ? S.n[0] : S.n[0] * S.n[1]);
    const long long total = (long long)(S.n[A] + 2) * S.n[(A + 1) % 3] * S.n[(A + 2) % 3];
    hipLaunchKernelGGL((k3_faces_line<real, A, OFF>), dim3((unsigned)((total - step + 63 - step) / (64 - step))), dim3(64), 0, st,
                       S);
}

template <typename real, int A, typename OFF>
static void launch_march(const Stage3<real> &S, hipStream_t st)
{
    const long long cols = (long long)S.n[0] * S.n[3 - A], groups = (cols + 63) / 64;  // of 64 columns
    if (S.n[0] * (A == 2 ? S.n[1] : 1) <= kLineStep || cols <= kLineCols) return launch_line<real, A, OFF>(S, st);
    const int len = march3(S.n, A, groups);
    const dim3 g((unsigned)(groups * ((S.n[A] + len) / len)));
    hipLaunchKernelGGL((k3_faces_march<real, A, OFF>), g, dim3(64), 0, st, S, len);
}

template <typename real, typename OFF>
static void launch_top2(const Stage3<real> &S, hipStream_t st)
{
    launch_line<real, 0, OFF>(S, st);
    launch_march<real, 1, OFF>(S, st);
    launch_march<real, 2, OFF>(S, st);
}

template <typename real, int R>
static void launch_faces_top(const Stage3<real> &S, hipStream_t st)
{
    if constexpr (R == 2) {
        // byte offsets into a variable of 4 GiB or more take 64 bits: in FP64 only, since face
        // ids of 31 bits (gpm3_create) end at 699 million cells, 2.8 GB a variable in FP32
        if constexpr (sizeof(real) == 8) {
            if ((unsigned long long)S.n[0] * S.n[1] * S.n[2] * sizeof(real) > 0xffffffffull)
                return launch_top2<real, size_t>(S, st);
        }
        launch_top2<real, unsigned>(S, st);
    } else {
        for (int a = 0; a < 3; ++a) {
            const long long nfa = (long long)(S.n[0] + (a == 0)) * (S.n[1] + (a == 1)) * (S.n[2] + (a == 2));
            const dim3 g((unsigned)((nfa + 127) / 128)), t(128);
            if (a == 0) hipLaunchKernelGGL((k3_faces_top<real, 0>), g, t, 0, st, S);
            if (a == 1) hipLaunchKernelGGL((k3_faces_top<real, 1>), g, t, 0, st, S);
            if (a == 2) hipLaunchKernelGGL((k3_faces_top<real, 2>), g, t, 0, st, S);
        }
    }
}

// Face id of axis a at cell (i, j, k) (the - face; + face: the next index along a).
template <typename real>
__device__ __forceinline__ int face3_id(const Stage3<real> &S, int a, int i, int j, int k)
{
    const int m0 = S.n[0] + (a == 0), m1 = S.n[1] + (a == 1);
    return S.fofs[a] + (k * m1 + j) * m0 + i;
}

template <typename real>
__device__ __forceinline__ void claims3(const Stage3<real> &S, const PassOut3 &P, int i, int j, int k, bool act)
{
    int fid[9];
    bool fok[9];
    const int c3[3] = {i, j, k};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int ip = i + (a == 0), jp = j + (a == 1), kp = k + (a == 2);
        fid[2 * a] = face3_id(S, a, i, j, k);
        fid[2 * a + 1] = face3_id(S, a, ip, jp, kp);
        fok[2 * a] = fok[2 * a + 1] = true;
        // periodic axis: the boundary face has a second copy at the other end
        const bool lo = c3[a] == 0, hi = c3[a] == S.n[a] - 1;
        fok[6 + a] = S.bc[a] == 0 && (lo || hi);
        const int e = lo ? S.n[a] : 0;
        fid[6 + a] = fok[6 + a] ? face3_id(S, a, a == 0 ? e : i, a == 1 ? e : j, a == 2 ? e : k) : fid[2 * a];
    }
    int cid[7];
    bool cok[7];
#pragma unroll
    for (int m = 0; m < 7; ++m) {
        const int ii = i + kBall[m][0], jj = j + kBall[m][1], kk = k + kBall[m][2];
        cok[m] = (S.bc[0] == 0 || (ii >= 0 && ii < S.n[0])) && (S.bc[1] == 0 || (jj >= 0 && jj < S.n[1])) &&
                 (S.bc[2] == 0 || (kk >= 0 && kk < S.n[2]));
        cid[m] = cok[m] ? (int)cell3(S, ii, jj, kk) : (int)cell3(S, i, j, k);
    }
    bool fmine[9], cmine[7];
    int nmine = 0;
    if (act) {
        unsigned fo[9], co[7];
#pragma unroll
        for (int m = 0; m < 9; ++m) fo[m] = atomicMax(&S.fstamp[fid[m]], fok[m] ? P.stamp : 0u);
#pragma unroll
        for (int m = 0; m < 7; ++m) co[m] = atomicMax(&S.cstamp[cid[m]], cok[m] ? P.stamp : 0u);
#pragma unroll
        for (int m = 0; m < 9; ++m) {
            fmine[m] = fok[m] && fo[m] < P.stamp;
            nmine += fmine[m] ? 1 : 0;
        }
#pragma unroll
        for (int m = 0; m < 7; ++m) {
            cmine[m] = cok[m] && co[m] < P.stamp;
            nmine += cmine[m] ? 65536 : 0;
        }
    } else {
#pragma unroll
        for (int m = 0; m < 9; ++m) fmine[m] = false;
#pragma unroll
        for (int m = 0; m < 7; ++m) cmine[m] = false;
    }
    int fb, cb;
    wave_reserve2(nmine, P.fcount, P.ccount, fb, cb);
    if (nmine != 0) {
#pragma unroll
        for (int m = 0; m < 9; ++m)
            if (fmine[m]) P.flist[fb++] = fid[m];
#pragma unroll
        for (int m = 0; m < 7; ++m)
            if (cmine[m]) P.clist[cb++] = cid[m];
    }
}

template <typename real>
__device__ __forceinline__ bool troubled3(const Stage3<real> &S0, int o, const real (&ust)[5], bool rs,
                                          const real (&r7)[7], int i, int j, int k)
{
    if (o == 0) return false;
    const Stage3<real> &S = *(const Stage3<real> *)reread((cptr<Stage3<real>>)&S0);
    const size_t plane = (size_t)S.n[0] * S.n[1] * S.n[2];
    const real g = S.gamma;
    const real rho = ust[0], p = p3(g, ust);
    if (!(finite(rho) && finite(p))) return true;
    if ((S.flags & 8u) && rs) return true;
    if (!(rho > real(0) && p > real(0))) return true;
    real lo = r7[0], hi = r7[0];
#pragma unroll
    for (int m = 1; m < 7; ++m) {
        lo = vmin(lo, r7[m]);
        hi = vmax(hi, r7[m]);
    }
    if (lo <= rho && rho <= hi) return false;                   // DMP
    if ((S.flags & 2u) && (hi - lo) < S.plat_thr) return false;  // plateau
    if (S.flags & 1u) {                                          // CSD
        real divV = real(0), gradp = real(0);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            real qp[5], qm[5];
            const size_t cp = cell3(S, i + (a == 0), j + (a == 1), k + (a == 2));
            const size_t cm = cell3(S, i - (a == 0), j - (a == 1), k - (a == 2));
#pragma unroll
            for (int v = 0; v < 5; ++v) {
                qp[v] = S.Us[v * plane + cp];
                qm[v] = S.Us[v * plane + cm];
            }
            divV = divV + (qp[1 + a] / qp[0] - qm[1 + a] / qm[0]) / (real(2) * S.d[a]);
            const real pp = p3(g, qp), pm = p3(g, qm);
            gradp = gradp + fabs(pp - pm) / (real(2) * S.d[a] * vmin(pp, pm));
        }
        if (divV >= -S.sigma_v && gradp <= S.sigma_p) return false;
    }
    if (S.flags & 4u) {  // u2
        real r25[25];
#pragma unroll
        for (int m = 0; m < 25; ++m)
            r25[m] = m < 7 ? r7[m] : S.Us[cell3(S, i + kBall[m][0], j + kBall[m][1], k + kBall[m][2])];
        // index in kBall of the offset (di, dj, dk) with |di|+|dj|+|dk| <= 2
        auto at = [&](int di, int dj, int dk) {
            int r = 0;
#pragma unroll
            for (int m = 0; m < 25; ++m)
                if (kBall[m][0] == di && kBall[m][1] == dj && kBall[m][2] == dk) r = m;
            return r25[r];
        };
        bool ok = true;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            real cmin = real(0), cmax = real(0);
#pragma unroll
            for (int m = 0; m < 7; ++m) {
                const int mi = kBall[m][0], mj = kBall[m][1], mk = kBall[m][2];
                real kap = S.curv[d][0] * at(mi, mj, mk);
                int slot = 2;
#pragma unroll
                for (int e = 0; e < 3; ++e) {
                    const int ex = e == 0, ey = e == 1, ez = e == 2;
                    const real pair = at(mi + ex, mj + ey, mk + ez) + at(mi - ex, mj - ey, mk - ez);
                    if (e == d) kap = fma(S.curv[d][1], pair, kap);
                    else kap = fma(S.curv[d][slot++], pair, kap);
                }
                if (m == 0) {
                    cmin = kap;
                    cmax = kap;
                } else {
                    cmin = vmin(cmin, kap);
                    cmax = vmax(cmax, kap);
                }
            }
            const bool pr = cmin * cmax > -S.delta;
            const bool a_ = pr && vmax(fabs(cmax), fabs(cmin)) < S.delta;
            const bool b_ = pr && fabs(cmin) >= real(0.5) * fabs(cmax);
            ok = ok && (a_ || b_);
        }
        if (ok) return false;
    }
    return true;
}

// ALL: the first evaluation, every cell at the top radius.  Bound by memory: each flux is
// read by the two cells of its face, so blocks go in runs to the XCDs, whose L2 then serves
// the second.  The arguments are read again where they are used (held from the kernel's
// entry they were moved to and from vector lanes, 600 instructions), the 18 outer cells of
// the density ball only where u2 is reached, and the claims run only in a wavefront with a
// lowered cell.  Measured: 192^3 FP32 322 -> 175 us (870 MB at least, 5.0 TB/s), 97 x 64 x
// 81 FP64 47 -> 30 us.
template <typename real, bool ALL>
__global__ __launch_bounds__(128) void k3_cells(const Stage3<real>, const int *list, const int *count, PassOut3 P)
{
    const Stage3<real> &S = first_arg<Stage3<real>>();
    auto again = [&]() -> const Stage3<real> & { return *(const Stage3<real> *)reread((cptr<Stage3<real>>)&S); };
    const int nc = S.n[0] * S.n[1] * S.n[2];
    int n = ALL ? nc : *count;
    n = n < nc ? n : nc;
    const int block = ALL ? xcd_tile(blockIdx.x, gridDim.x) : (int)blockIdx.x;
    if (n <= block * (int)blockDim.x) return;
    P.stamp = *S.stamp0 + P.stamp;  // P.stamp carries the pass index
    const size_t plane = (size_t)nc;
    const real dt = (real)(*S.dt);
    const int stride = gridDim.x * blockDim.x;
    const int nround = (n + stride - 1) / stride;
    for (int r = 0; r < nround; ++r) {
        const int idx = r * stride + block * blockDim.x + threadIdx.x;
        bool tr = false;
        int i = 0, j = 0, k = 0;
        if (idx < n) {
            const int c = ALL ? idx : list[idx];
            const Stage3<real> &G = again();
            i = c % G.n[0];
            const int jk = c / G.n[0];
            j = jk % G.n[1];
            k = jk / G.n[1];
            real ust[5];
            real div[5] = {real(0), real(0), real(0), real(0), real(0)};
            // every flux, flag and state value of the cell loaded first, then one
            // wait (the flag tests and the divisions had split the loads by axis)
            real fpv[3][5], fmv[3][5], us[5], r7[7];
            int fl = 0;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const Stage3<real> &H = again();
                const int m0 = H.n[0] + (a == 0), m1 = H.n[1] + (a == 1), m2 = H.n[2] + (a == 2);
                const size_t nfa = (size_t)m0 * m1 * m2;
                const int fm = (k * m1 + j) * m0 + i;
                const int fp = ((k + (a == 2)) * m1 + j + (a == 1)) * m0 + i + (a == 0);
#pragma unroll
                for (int v = 0; v < 5; ++v) {
                    fpv[a][v] = H.F[a][v * nfa + fp];
                    fmv[a][v] = H.F[a][v * nfa + fm];
                }
                fl |= H.Ff[a][fm] | H.Ff[a][fp];  // either side of either face
            }
            const Stage3<real> &V = again();
#pragma unroll
            for (int v = 0; v < 5; ++v) us[v] = V.Us[v * plane + c];
            r7[0] = us[0];
#pragma unroll
            for (int m = 1; m < 7; ++m) r7[m] = V.Us[cell3(V, i + kBall[m][0], j + kBall[m][1], k + kBall[m][2])];
            const int o = ALL ? V.top : V.order[c];
            __builtin_amdgcn_sched_barrier(0);
            const bool rs = fl != 0;
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int v = 0; v < 5; ++v) div[v] = div[v] + (fpv[a][v] - fmv[a][v]) / V.d[a];
#pragma unroll
            for (int v = 0; v < 5; ++v) ust[v] = us[v] - dt * div[v];
            tr = troubled3(S, o, ust, rs, r7, i, j, k);
            const Stage3<real> &W = again();
#pragma unroll
            for (int v = 0; v < 5; ++v) {
                const real un = W.s == 0 ? real(0) : W.Un[v * plane + c];
                W.Uout[v * plane + c] = combine(W.s, un, ust[v]);
            }
            if (ALL || tr)
                W.order[c] = (uint8_t)(tr ? next_radius(W.next[0], W.next[1], W.next[2], W.next[3], o) : o);
        }
        wave_count(tr, P.tcount);
        if (__ballot(tr) != 0ull) claims3(again(), P, i, j, k, tr);
    }
}

__global__ void k3_reset(Ctl *ctl, int nzero, unsigned stamp0)
{
    for (int k = threadIdx.x; k < nzero && k < kMaxPasses + 2; k += blockDim.x) {
        ctl->nface[k] = 0;
        ctl->ncell[k] = 0;
        ctl->ntroub[k] = 0;
    }
    if (threadIdx.x == 0) ctl->stamp0 = stamp0;
}

// Four cells a thread and round, their 20 loads issued before the arithmetic (the maximum
// does not depend on the order): one at a time each waited for its loads and, with one cell
// a thread, the block's reduction was most of the work (97 x 64 x 81 FP64: 20.0 -> 8.7 us,
// 192^3 FP32: 46 -> 41 us; read once at 5.1 TB/s they take 4 and 28).
template <typename real>
__global__ __launch_bounds__(256) void k3_dt(const real *U, size_t n, double gamma, double dx, double dy, double dz,
                                             unsigned long long *lam_bits)
{
    __shared__ double red[256];
    constexpr int kU = 4;
    double lam = 0.0;
    const size_t first = (size_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (size_t)gridDim.x * blockDim.x;
    for (size_t t0 = first; t0 < n; t0 += kU * stride) {
        real q[kU][5];
#pragma unroll
        for (int m = 0; m < kU; ++m) {
            const size_t t = t0 + (size_t)m * stride, tt = t < n ? t : first;  // in bounds; skipped below
#pragma unroll
            for (int v = 0; v < 5; ++v) q[m][v] = U[(size_t)v * n + tt];
        }
#pragma unroll
        for (int m = 0; m < kU; ++m) {
            if (t0 + (size_t)m * stride >= n) continue;
            const double r = q[m][0], mx = q[m][1], my = q[m][2], mz = q[m][3], E = q[m][4];
            const double p = (gamma - 1.0) * (E - 0.5 * (mx * mx + my * my + mz * mz) / r);
            if (!(r > 0.0 && p > 0.0 && __builtin_isfinite(r) && __builtin_isfinite(p))) continue;
            const double cs = sqrt(gamma * p / r);
            const double lx = (fabs(mx / r) + cs) / dx, ly = (fabs(my / r) + cs) / dy, lz = (fabs(mz / r) + cs) / dz;
            double l = lx > ly ? lx : ly;
            l = lz > l ? lz : l;
            lam = l > lam ? l : lam;
        }
    }
    red[threadIdx.x] = lam;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] = red[threadIdx.x] > red[threadIdx.x + s] ? red[threadIdx.x] : red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0 && red[0] > 0.0) {
        // as in 2D: no atomic from a block whose value cannot raise the maximum
        const unsigned long long b = (unsigned long long)__double_as_longlong(red[0]);
        if (b > __hip_atomic_load(lam_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(lam_bits, b);
    }
}

__global__ void k3_dt_begin(Ctl *ctl) { ctl->lam_bits = 0ull; }
__global__ void k3_dt_end(Ctl *ctl, double cfl) { ctl->dt = cfl / __longlong_as_double((long long)ctl->lam_bits); }

__global__ __launch_bounds__(256) void k3_hist(const uint8_t *order, size_t n, int l0, int l1, int l2,
                                               unsigned long long *cnt)
{
    __shared__ unsigned long long c[3];
    if (threadIdx.x < 3) c[threadIdx.x] = 0ull;
    __syncthreads();
    for (size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += (size_t)gridDim.x * blockDim.x) {
        const int o = order[t];
        const int l = o == 2 ? l2 : (o == 1 ? l1 : l0);
        atomicAdd(&c[l], 1ull);
    }
    __syncthreads();
    if (threadIdx.x < 3 && c[threadIdx.x]) atomicAdd(&cnt[threadIdx.x], c[threadIdx.x]);
}

// Compensated (double-double) totals, block partials then a fixed-order sum.
template <typename real>
__global__ __launch_bounds__(256) void k3_tot_partial(const real *U, size_t n, double *partial)
{
    __shared__ double sh[256], sl[256];
    const int v = blockIdx.y;
    double hi = 0.0, lo = 0.0;
    for (size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += (size_t)gridDim.x * blockDim.x) {
        const double x = (double)U[v * n + t];
        const double s = hi + x, bb = s - hi, e = (hi - (s - bb)) + (x - bb);
        lo += e;
        hi = s;
    }
    sh[threadIdx.x] = hi;
    sl[threadIdx.x] = lo;
    __syncthreads();
    if (threadIdx.x == 0) {
        double H = 0.0, L = 0.0;
        for (int k = 0; k < 256; ++k) {
            const double s = H + sh[k], bb = s - H, e = (H - (s - bb)) + (sh[k] - bb);
            L += e + sl[k];
            H = s;
        }
        partial[(size_t)v * gridDim.x * 2 + 2 * blockIdx.x] = H;
        partial[(size_t)v * gridDim.x * 2 + 2 * blockIdx.x + 1] = L;
    }
}

__global__ void k3_tot_final(const double *partial, int nblk, double vol, double *tot)
{
    const int v = threadIdx.x;
    if (v >= 5) return;
    double H = 0.0, L = 0.0;
    for (int b = 0; b < nblk; ++b) {
        const double x = partial[(size_t)v * nblk * 2 + 2 * b];
        const double s = H + x, bb = s - H, e = (H - (s - bb)) + (x - bb);
        L += e + partial[(size_t)v * nblk * 2 + 2 * b + 1];
        H = s;
    }
    tot[v] = (H + L) * vol;
}

}  // namespace gpm

using namespace gpm;

// ------------------------------------------------------------------- host side
namespace {

constexpr size_t kAl = 256;
size_t al(size_t x) { return (x + kAl - 1) / kAl * kAl; }
constexpr int kTot3Blocks = 1024;

}  // namespace

struct gpm3_ctx {
    gpm_grid grid;
    int prec;
    hipStream_t stream;
    int n[3];
    size_t ncell, nface[3], nfaces;
    double d[3];
    bool have_scheme = false;
    gpm_scheme scheme;
    int top = 0, next[4] = {0, 0, 0, 0}, levidx[3] = {0, 0, 0};
    std::vector<double> z64, qw64, pz64;
    std::vector<float> z32, qw32, pz32;
    double curv64[3][4];
    float curv32[3][4];
    char *state = nullptr, *work = nullptr;
    int cur = 0;
    uint8_t *order = nullptr;
    unsigned *cstamp = nullptr, *fstamp = nullptr;
    int *flist[2] = {nullptr, nullptr}, *clist[2] = {nullptr, nullptr};
    void *F[3] = {nullptr, nullptr, nullptr};
    uint8_t *Ff[3] = {nullptr, nullptr, nullptr};
    Ctl *ctl = nullptr;
    double *partial = nullptr;
    void *wtab = nullptr;  // z then qw, context precision
    unsigned pass = 0;
    int last_npass = 0;
    bool fresh = true;
    int *pinned = nullptr;
    std::string err;
};

static gpm_status f3(gpm3_ctx *c, gpm_status st, const std::string &m)
{
    if (c) c->err = m;
    return st;
}

#define H3(c, expr)                                                                        \
    do {                                                                                   \
        hipError_t e_ = (expr);                                                            \
        if (e_ != hipSuccess) return f3((c), GPM_EHIP, std::string(#expr) + ": " + hipGetErrorString(e_)); \
    } while (0)

static size_t esz3(const gpm3_ctx *c) { return c->prec == GPM_F64 ? 8 : 4; }
static size_t slot3(const gpm3_ctx *c) { return al(5 * c->ncell * esz3(c)); }

enum { X_ORDER, X_CST, X_FST, X_FL0, X_FL1, X_CL0, X_CL1, X_F0, X_F1, X_F2, X_FF0, X_FF1, X_FF2, X_CTL, X_PART, X_W, X_N };

static size_t layout3(const gpm3_ctx *c, size_t off[X_N])
{
    const size_t e = esz3(c);
    const size_t sz[X_N] = {c->ncell, 4 * c->ncell, 4 * c->nfaces, 4 * c->nfaces, 4 * c->nfaces, 4 * c->ncell,
                            4 * c->ncell, 5 * e * c->nface[0], 5 * e * c->nface[1], 5 * e * c->nface[2],
                            c->nface[0], c->nface[1], c->nface[2], sizeof(Ctl),
                            ((size_t)kTot3Blocks * 5 * 2 + 8) * sizeof(double), (size_t)(2 * kZ3 + 2 * 9 + kPZ3) * e};
    size_t o = 0;
    for (int k = 0; k < X_N; ++k) {
        off[k] = o;
        o = al(o + sz[k]);
    }
    return o;
}

static void *slotp(gpm3_ctx *c, int s) { return c->state + (size_t)s * slot3(c); }

template <typename real>
static Stage3<real> args3(gpm3_ctx *c, int s, const void *Un, const void *Us, void *Uout)
{
    Stage3<real> S;
    S.Un = (const real *)Un;
    S.Us = (const real *)Us;
    S.Uout = (real *)Uout;
    S.dt = &c->ctl->dt;
    S.order = c->order;
    for (int a = 0; a < 3; ++a) {
        S.F[a] = (real *)c->F[a];
        S.Ff[a] = c->Ff[a];
        S.n[a] = c->n[a];
        S.bc[a] = c->grid.bc[a];
        S.d[a] = (real)c->d[a];
    }
    S.fofs[0] = 0;
    S.fofs[1] = (int)c->nface[0];
    S.fofs[2] = (int)(c->nface[0] + c->nface[1]);
    S.fofs[3] = (int)c->nfaces;
    S.cstamp = c->cstamp;
    S.fstamp = c->fstamp;
    S.s = s;
    S.top = c->top;
    S.flags = c->scheme.flags;
    for (int r = 0; r < 4; ++r) S.next[r] = c->next[r];
    S.gamma = (real)c->grid.gamma;
    S.sigma_v = (real)c->scheme.sigma_v;
    S.sigma_p = (real)c->scheme.sigma_p;
    double d3 = 1e300, dm = 1e300;
    for (int a = 0; a < 3; ++a) {
        d3 = c->d[a] * c->d[a] * c->d[a] < d3 ? c->d[a] * c->d[a] * c->d[a] : d3;
        dm = c->d[a] < dm ? c->d[a] : dm;
    }
    S.plat_thr = (real)d3;
    S.delta = (real)dm;
    S.z = (const real *)c->wtab;
    S.qw = (const real *)c->wtab + 2 * kZ3;
    S.pz = (const real *)c->wtab + 2 * kZ3 + 18;
    for (int d = 0; d < 3; ++d)
        for (int k = 0; k < 4; ++k) S.curv[d][k] = sizeof(real) == 8 ? (real)c->curv64[d][k] : (real)c->curv32[d][k];
    S.stamp0 = &c->ctl->stamp0;
    return S;
}

template <typename real>
static gpm_status stage3(gpm3_ctx *c, int s, const void *Un, const void *Us, void *Uout)
{
    Stage3<real> S = args3<real>(c, s, Un, Us, Uout);
    if (c->pass >= 0xffffffffu - (unsigned)(2 * kMaxPasses + 8)) {
        H3(c, hipMemsetAsync(c->cstamp, 0, 4 * c->ncell, c->stream));
        H3(c, hipMemsetAsync(c->fstamp, 0, 4 * c->nfaces, c->stream));
        c->pass = 0;
    }
    const unsigned stamp0 = c->pass + 1;
    c->pass += (unsigned)kMaxPasses + 2;
    const int nzero = c->fresh ? kMaxPasses + 2 : (c->last_npass + 3 < kMaxPasses + 2 ? c->last_npass + 3 : kMaxPasses + 2);
    c->fresh = false;
    hipLaunchKernelGGL(k3_reset, dim3(1), dim3(256), 0, c->stream, c->ctl, nzero, stamp0);
    // first evaluation: every face at the top radius, then every cell
    int nbc = (int)((c->ncell + 127) / 128);
    if (nbc > 65536) nbc = 65536;
    if (c->top == 2) launch_faces_top<real, 2>(S, c->stream);
    else launch_faces_top<real, 1>(S, c->stream);  // a scheme's top radius is 1 or 2
    PassOut3 P;
    P.flist = c->flist[1];
    P.clist = c->clist[1];
    P.fcount = &c->ctl->nface[1];
    P.ccount = &c->ctl->ncell[1];
    P.tcount = &c->ctl->ntroub[0];
    P.stamp = 0;
    hipLaunchKernelGGL((k3_cells<real, true>), dim3(nbc), dim3(128), 0, c->stream, S, (const int *)nullptr, (const int *)nullptr, P);
    H3(c, hipGetLastError());
    // cascade passes in batches, with a host check of the counts per batch
    int nb = (int)((c->ncell + 127) / 128);
    if (nb > 2048) nb = 2048;
    int k = 1, batch = 4;
    for (;;) {
        H3(c, hipMemcpyAsync(c->pinned, &c->ctl->ntroub[k - 1], sizeof(int), hipMemcpyDeviceToHost, c->stream));
        H3(c, hipStreamSynchronize(c->stream));
        if (*c->pinned == 0) break;
        if (k + batch > kMaxPasses) {
            c->last_npass = k - 1;
            return f3(c, GPM_ENOTCONV, "MOOD loop exceeded the pass limit");
        }
        for (int b = 0; b < batch; ++b, ++k) {
            hipLaunchKernelGGL(k3_faces<real>, dim3(nb), dim3(128), 0, c->stream, S, c->flist[k & 1], &c->ctl->nface[k]);
            PassOut3 Q;
            Q.flist = c->flist[(k + 1) & 1];
            Q.clist = c->clist[(k + 1) & 1];
            Q.fcount = &c->ctl->nface[k + 1];
            Q.ccount = &c->ctl->ncell[k + 1];
            Q.tcount = &c->ctl->ntroub[k];
            Q.stamp = (unsigned)k;
            hipLaunchKernelGGL((k3_cells<real, false>), dim3(nb), dim3(128), 0, c->stream, S, c->clist[k & 1], &c->ctl->ncell[k], Q);
        }
        H3(c, hipGetLastError());
        if (batch < 32) batch *= 2;
    }
    c->last_npass = k - 1;
    return GPM_OK;
}

template <typename real>
static gpm_status dt3(gpm3_ctx *c, const void *U, double cfl)
{
    hipLaunchKernelGGL(k3_dt_begin, dim3(1), dim3(1), 0, c->stream, c->ctl);
    size_t nblk = (c->ncell + 1023) / 1024;  // four cells a thread
    if (nblk > 4096) nblk = 4096;
    hipLaunchKernelGGL(k3_dt<real>, dim3((unsigned)nblk), dim3(256), 0, c->stream, (const real *)U, c->ncell,
                       c->grid.gamma, c->d[0], c->d[1], c->d[2], &c->ctl->lam_bits);
    hipLaunchKernelGGL(k3_dt_end, dim3(1), dim3(1), 0, c->stream, c->ctl, cfl);
    H3(c, hipGetLastError());
    return GPM_OK;
}

extern "C" {

gpm_status gpm3_create(const gpm_grid *grid, int prec, void *hip_stream, gpm3_ctx **out)
{
    if (!grid || !out) return GPM_EINVAL;
    *out = nullptr;
    if (grid->dim != 3) return GPM_EUNSUPPORTED;
    if (prec != GPM_F32 && prec != GPM_F64) return GPM_EINVAL;
    size_t ncell = 1;
    for (int a = 0; a < 3; ++a) {
        if (grid->n[a] < 1 || grid->n[a] > 4096) return GPM_EINVAL;
        if (!(grid->hi[a] > grid->lo[a])) return GPM_EINVAL;
        if (grid->bc[a] == GPM_BC_REFLECT || grid->slit != 0) return GPM_EUNSUPPORTED;  // 2D only
        if (grid->bc[a] != GPM_BC_PERIODIC && grid->bc[a] != GPM_BC_OUTFLOW) return GPM_EINVAL;
        if (grid->bc[a] == GPM_BC_PERIODIC && grid->n[a] < 3) return GPM_EUNSUPPORTED;
        ncell *= (size_t)grid->n[a];
    }
    if (!(grid->gamma > 1.0)) return GPM_EINVAL;
    if (3 * ncell + 3 * 4096 * 4096 > 0x7fffffffull) return GPM_EUNSUPPORTED;  // 32-bit face ids
    gpm3_ctx *c = new (std::nothrow) gpm3_ctx;
    if (!c) return GPM_ENOMEM;
    c->grid = *grid;
    c->prec = prec;
    c->stream = (hipStream_t)hip_stream;
    for (int a = 0; a < 3; ++a) {
        c->n[a] = grid->n[a];
        c->d[a] = (grid->hi[a] - grid->lo[a]) / grid->n[a];
    }
    c->ncell = ncell;
    c->nfaces = 0;
    for (int a = 0; a < 3; ++a) {
        c->nface[a] = (size_t)(c->n[0] + (a == 0)) * (c->n[1] + (a == 1)) * (c->n[2] + (a == 2));
        c->nfaces += c->nface[a];
    }
    if (hipHostMalloc((void **)&c->pinned, 64, hipHostMallocDefault) != hipSuccess) {
        delete c;
        return GPM_EHIP;
    }
    *out = c;
    return GPM_OK;
}

void gpm3_destroy(gpm3_ctx *c)
{
    if (!c) return;
    if (c->pinned) (void)hipHostFree(c->pinned);
    delete c;
}

const char *gpm3_last_error(const gpm3_ctx *c) { return c ? c->err.c_str() : ""; }

static gpm_status upload3(gpm3_ctx *c)
{
    if (!c->wtab || !c->have_scheme) return GPM_OK;
    const size_t e = esz3(c);
    std::vector<char> buf((2 * kZ3 + 18 + kPZ3) * e);
    if (e == 8) {
        std::memcpy(buf.data(), c->z64.data(), 2 * kZ3 * 8);
        std::memcpy(buf.data() + 2 * kZ3 * 8, c->qw64.data(), 18 * 8);
        std::memcpy(buf.data() + (2 * kZ3 + 18) * 8, c->pz64.data(), kPZ3 * 8);
    } else {
        std::memcpy(buf.data(), c->z32.data(), 2 * kZ3 * 4);
        std::memcpy(buf.data() + 2 * kZ3 * 4, c->qw32.data(), 18 * 4);
        std::memcpy(buf.data() + (2 * kZ3 + 18) * 4, c->pz32.data(), kPZ3 * 4);
    }
    H3(c, hipMemcpyAsync(c->wtab, buf.data(), buf.size(), hipMemcpyHostToDevice, c->stream));
    H3(c, hipStreamSynchronize(c->stream));
    return GPM_OK;
}

gpm_status gpm3_set_scheme(gpm3_ctx *c, const gpm_scheme *s)
{
    if (!c || !s) return GPM_EINVAL;
    if (s->nlev < 1 || s->nlev > 3) return f3(c, GPM_EINVAL, "nlev must be 1..3");
    if (s->stencil != GPM_STENCIL_DIAMOND) return f3(c, GPM_EUNSUPPORTED, "the 3D engine uses the L1-ball stencil");
    if (s->solver != GPM_SOLVER_HLLC) return f3(c, GPM_EUNSUPPORTED, "the 3D engine uses HLLC");
    for (int l = 0; l < s->nlev; ++l) {
        if (s->radius[l] < 0 || s->radius[l] > 2) return f3(c, GPM_EINVAL, "3D radius must be 0..2");
        if (l > 0 && !(s->radius[l] < s->radius[l - 1])) return f3(c, GPM_EINVAL, "cascade must strictly decrease");
    }
    if (s->radius[s->nlev - 1] != 0) return f3(c, GPM_EINVAL, "cascade must end at radius 0 (FOG)");
    if (s->radius[0] == 0) return f3(c, GPM_EINVAL, "top scheme must have radius >= 1");
    if (!(s->ell >= 0.0)) return f3(c, GPM_EINVAL, "ell must be >= 0");
    double dmin = c->d[0] < c->d[1] ? c->d[0] : c->d[1];
    dmin = c->d[2] < dmin ? c->d[2] : dmin;
    const double ell = s->ell > 0.0 ? s->ell : 12.0 * dmin;
    c->z64.assign(2 * kZ3, 0.0);
    c->z32.assign(2 * kZ3, 0.0f);
    c->qw64.assign(18, 0.0);
    c->qw32.assign(18, 0.0f);
    c->pz64.assign(kPZ3, 0.0);
    c->pz32.assign(kPZ3, 0.0f);
    for (int R = 1; R <= 2; ++R) {
        bool used = false;
        for (int l = 0; l < s->nlev; ++l) used = used || s->radius[l] == R;
        if (!used) continue;
        Gpw3Level L;
        if (gpw3_level(R, ell / c->d[0], ell / c->d[1], ell / c->d[2], &L) != 0)
            return f3(c, GPM_EINVAL, "GP covariance matrix not positive definite");
        for (int f = 0; f < 6; ++f)
            for (int k = 0; k < L.nq; ++k)
                for (int m = 0; m < kNBall[R]; ++m) {
                    const size_t o = ((size_t)(R - 1) * 6 + f) * 9 * 25 + k * 25 + m;
                    c->z64[o] = L.z64[f][k][m];
                    c->z32[o] = L.z32[f][k][m];
                }
        for (int k = 0; k < L.nq; ++k) {
            c->qw64[(R - 1) * 9 + k] = L.qw64[k];
            c->qw32[(R - 1) * 9 + k] = L.qw32[k];
        }
        if (R == 2)
            for (int f = 0; f < 6; ++f)
                for (int cls = 0; cls < 4; ++cls)
                    for (int e = 0; e < kNPar3; ++e) {
                        c->pz64[((size_t)f * 4 + cls) * kNPar3 + e] = L.pz64[f][cls][e];
                        c->pz32[((size_t)f * 4 + cls) * kNPar3 + e] = L.pz32[f][cls][e];
                    }
    }
    Gpw3Curv K;
    if (gpw3_curvature(ell / c->d[0], ell / c->d[1], ell / c->d[2], ell, &K) != 0)
        return f3(c, GPM_EINVAL, "GP-R1 covariance matrix not positive definite");
    std::memcpy(c->curv64, K.w64, sizeof(c->curv64));
    std::memcpy(c->curv32, K.w32, sizeof(c->curv32));
    c->scheme = *s;
    c->scheme.ell = ell;
    c->top = s->radius[0];
    for (int r = 0; r < 4; ++r) c->next[r] = 0;
    for (int l = 0; l < s->nlev; ++l) {
        c->levidx[s->radius[l]] = l;
        c->next[s->radius[l]] = l + 1 < s->nlev ? s->radius[l + 1] : 0;
    }
    c->have_scheme = true;
    return upload3(c);
}

gpm_status gpm3_workspace_size(const gpm3_ctx *c, size_t *state_bytes, size_t *work_bytes)
{
    if (!c) return GPM_EINVAL;
    size_t off[X_N];
    if (state_bytes) *state_bytes = 3 * slot3(c);
    if (work_bytes) *work_bytes = layout3(c, off);
    return GPM_OK;
}

gpm_status gpm3_bind(gpm3_ctx *c, void *state, void *work)
{
    if (!c || !state || !work) return GPM_EINVAL;
    if (((uintptr_t)state % kAl) || ((uintptr_t)work % kAl)) return f3(c, GPM_EINVAL, "buffers must be 256-byte aligned");
    size_t off[X_N];
    const size_t wb = layout3(c, off);
    c->state = (char *)state;
    c->work = (char *)work;
    c->order = (uint8_t *)(c->work + off[X_ORDER]);
    c->cstamp = (unsigned *)(c->work + off[X_CST]);
    c->fstamp = (unsigned *)(c->work + off[X_FST]);
    c->flist[0] = (int *)(c->work + off[X_FL0]);
    c->flist[1] = (int *)(c->work + off[X_FL1]);
    c->clist[0] = (int *)(c->work + off[X_CL0]);
    c->clist[1] = (int *)(c->work + off[X_CL1]);
    for (int a = 0; a < 3; ++a) {
        c->F[a] = c->work + off[X_F0 + a];
        c->Ff[a] = (uint8_t *)(c->work + off[X_FF0 + a]);
    }
    c->ctl = (Ctl *)(c->work + off[X_CTL]);
    c->partial = (double *)(c->work + off[X_PART]);
    c->wtab = c->work + off[X_W];
    c->cur = 0;
    c->pass = 0;
    c->fresh = true;
    H3(c, hipMemsetAsync(c->work, 0, wb, c->stream));
    H3(c, hipStreamSynchronize(c->stream));
    return upload3(c);
}

gpm_status gpm3_init_state(gpm3_ctx *c, const double *U)
{
    if (!c || !U) return GPM_EINVAL;
    if (!c->state) return f3(c, GPM_ESTATE, "not bound");
    const size_t n = 5 * c->ncell;
    if (c->prec == GPM_F64) {
        H3(c, hipMemcpyAsync(slotp(c, c->cur), U, n * 8, hipMemcpyHostToDevice, c->stream));
        H3(c, hipStreamSynchronize(c->stream));
    } else {
        std::vector<float> t(n);
        for (size_t k = 0; k < n; ++k) t[k] = (float)U[k];
        H3(c, hipMemcpyAsync(slotp(c, c->cur), t.data(), n * 4, hipMemcpyHostToDevice, c->stream));
        H3(c, hipStreamSynchronize(c->stream));
    }
    return GPM_OK;
}

gpm_status gpm3_get_state(gpm3_ctx *c, double *U)
{
    if (!c || !U) return GPM_EINVAL;
    if (!c->state) return f3(c, GPM_ESTATE, "not bound");
    const size_t n = 5 * c->ncell;
    if (c->prec == GPM_F64) {
        H3(c, hipMemcpyAsync(U, slotp(c, c->cur), n * 8, hipMemcpyDeviceToHost, c->stream));
        H3(c, hipStreamSynchronize(c->stream));
    } else {
        std::vector<float> t(n);
        H3(c, hipMemcpyAsync(t.data(), slotp(c, c->cur), n * 4, hipMemcpyDeviceToHost, c->stream));
        H3(c, hipStreamSynchronize(c->stream));
        for (size_t k = 0; k < n; ++k) U[k] = t[k];
    }
    return GPM_OK;
}

gpm_status gpm3_compute_dt(gpm3_ctx *c, double cfl, double *dt_host)
{
    if (!c) return GPM_EINVAL;
    if (!c->state) return f3(c, GPM_ESTATE, "not bound");
    if (!(cfl > 0.0)) return f3(c, GPM_EINVAL, "cfl must be > 0");
    gpm_status st = c->prec == GPM_F64 ? dt3<double>(c, slotp(c, c->cur), cfl) : dt3<float>(c, slotp(c, c->cur), cfl);
    if (st != GPM_OK) return st;
    if (dt_host) {
        H3(c, hipMemcpyAsync(dt_host, &c->ctl->dt, sizeof(double), hipMemcpyDeviceToHost, c->stream));
        H3(c, hipStreamSynchronize(c->stream));
    }
    return GPM_OK;
}

gpm_status gpm3_step(gpm3_ctx *c, double cfl, int nsteps)
{
    if (!c || nsteps < 0) return GPM_EINVAL;
    if (!c->have_scheme) return f3(c, GPM_ESTATE, "no scheme set");
    if (!c->state) return f3(c, GPM_ESTATE, "not bound");
    if (!(cfl > 0.0)) return f3(c, GPM_EINVAL, "cfl must be > 0");
    for (int n = 0; n < nsteps; ++n) {
        const int u0 = c->cur, a = (c->cur + 1) % 3, b = (c->cur + 2) % 3;
        const bool dbl = c->prec == GPM_F64;
        gpm_status st = dbl ? dt3<double>(c, slotp(c, u0), cfl) : dt3<float>(c, slotp(c, u0), cfl);
        if (st == GPM_OK) st = dbl ? stage3<double>(c, 0, slotp(c, u0), slotp(c, u0), slotp(c, a))
                                   : stage3<float>(c, 0, slotp(c, u0), slotp(c, u0), slotp(c, a));
        if (st == GPM_OK) st = dbl ? stage3<double>(c, 1, slotp(c, u0), slotp(c, a), slotp(c, b))
                                   : stage3<float>(c, 1, slotp(c, u0), slotp(c, a), slotp(c, b));
        if (st == GPM_OK) st = dbl ? stage3<double>(c, 2, slotp(c, u0), slotp(c, b), slotp(c, a))
                                   : stage3<float>(c, 2, slotp(c, u0), slotp(c, b), slotp(c, a));
        if (st != GPM_OK) return st;
        c->cur = a;
    }
    return GPM_OK;
}

gpm_status gpm3_troubled_counts(gpm3_ctx *c, long long counts[3], int *mood_iters)
{
    if (!c) return GPM_EINVAL;
    if (!c->state) return f3(c, GPM_ESTATE, "not bound");
    H3(c, hipMemsetAsync(c->ctl->levcnt, 0, sizeof(c->ctl->levcnt), c->stream));
    hipLaunchKernelGGL(k3_hist, dim3(1024), dim3(256), 0, c->stream, c->order, c->ncell, c->levidx[0], c->levidx[1],
                       c->levidx[2], c->ctl->levcnt);
    unsigned long long lc[3];
    H3(c, hipMemcpyAsync(lc, c->ctl->levcnt, sizeof(lc), hipMemcpyDeviceToHost, c->stream));
    // passes are queued in batches: count those that had cells to re-evaluate
    std::vector<int> nc(c->last_npass + 2);
    H3(c, hipMemcpyAsync(nc.data(), c->ctl->ncell, sizeof(int) * nc.size(), hipMemcpyDeviceToHost, c->stream));
    H3(c, hipStreamSynchronize(c->stream));
    if (counts)
        for (int l = 0; l < 3; ++l) counts[l] = (long long)lc[l];
    if (mood_iters) {
        int it = 1;
        for (size_t k = 1; k < nc.size(); ++k)
            if (nc[k] > 0) ++it;
        *mood_iters = it;
    }
    return GPM_OK;
}

gpm_status gpm3_get_order_mask(gpm3_ctx *c, unsigned char *out)
{
    if (!c || !out) return GPM_EINVAL;
    if (!c->state) return f3(c, GPM_ESTATE, "not bound");
    H3(c, hipMemcpyAsync(out, c->order, c->ncell, hipMemcpyDeviceToHost, c->stream));
    H3(c, hipStreamSynchronize(c->stream));
    return GPM_OK;
}

gpm_status gpm3_totals(gpm3_ctx *c, double totals[5])
{
    if (!c || !totals) return GPM_EINVAL;
    if (!c->state) return f3(c, GPM_ESTATE, "not bound");
    const int nblk = kTot3Blocks;
    if (c->prec == GPM_F64)
        hipLaunchKernelGGL(k3_tot_partial<double>, dim3(nblk, 5), dim3(256), 0, c->stream,
                           (const double *)slotp(c, c->cur), c->ncell, c->partial);
    else
        hipLaunchKernelGGL(k3_tot_partial<float>, dim3(nblk, 5), dim3(256), 0, c->stream,
                           (const float *)slotp(c, c->cur), c->ncell, c->partial);
    double *tot = c->partial + (size_t)kTot3Blocks * 5 * 2;
    hipLaunchKernelGGL(k3_tot_final, dim3(1), dim3(64), 0, c->stream, c->partial, nblk, c->d[0] * c->d[1] * c->d[2],
                       tot);
    double t[5];
    H3(c, hipMemcpyAsync(t, tot, sizeof(t), hipMemcpyDeviceToHost, c->stream));
    H3(c, hipStreamSynchronize(c->stream));
    for (int v = 0; v < 5; ++v) totals[v] = t[v];
    return GPM_OK;
}

}  // extern "C"
