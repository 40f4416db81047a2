// HIP kernels of the 2D GP-MOOD stage for gfx950 (CDNA4).
//
// First pass (k_first_pass): every cell at the top order.  One 64-lane wavefront
// owns a strip of 62 columns (lanes 1..62; lanes 0 and 63 are the halo that
// supplies the neighbouring face states) and marches upward through `rows` rows.
// The stage input of rows j-3..j+4 sits in a per-wavefront ring of 8 LDS rows
// (70 columns x 4 variables), loaded once with coalesced row loads and the
// boundary conditions applied as index remaps.  At row j each lane reconstructs
// all 4q face states of its cell (eq. (gp_reconstructor) in the quarter basis),
// exchanges x-face states with its right neighbour by a lane shuffle, evaluates
// HLLC on its own x face, and evaluates the y face below it against the y+ states
// it kept from row j-1.  Cell (i, j-1) is then complete: candidate, detection,
// RK combine.  Every face flux (and its Riemann-state CAD flags) is stored for the
// cascade.  A troubled cell takes the next scheme of the cascade at once and is
// listed; a follow-up kernel claims its four faces and the five cells whose
// candidates they change.  No block barrier is needed: each wavefront only reads
// LDS it wrote itself.
//
// Cascade pass k (k_faces, then k_cells): recompute the claimed faces at their new
// EDP_1 order (min of the two cells' radii), then re-evaluate the claimed cells
// from the stored fluxes, re-detect, lower the troubled ones and claim the faces
// and cells of pass k+1.  Each face flux is computed once and read by both of its
// cells, so the update stays exactly conservative.  Every list holds each face or
// cell at most once (claim stamps), and both kernels read their item count from
// device memory and return at once when it is zero, so passes can be queued
// without a host round trip.
#include "gpmood_device.h"
#include "gpmood_index.h"
#include "gpmood_launch.h"

namespace gpm {

constexpr int LW = 70;  // LDS columns per ring row: 64 lanes + 3 halo columns each side

// One wavefront's strip (tile wid of the problem) of the first pass; ring is the
// wavefront's LDS ring.  ISO: A.iso is 1 (the y states read the x weights).
// A lowered cell is only appended to P.clist (count P.ccount); its claims are
// made after the pass (k_claims_first, or k_claims_first_batch in a batch), which keeps
// the claim atomics, and the wait for their results, out of the march.
template <typename real, int RT, bool ISO, bool HLL, bool BND>
__device__ __forceinline__ void first_pass_wave(const StageArgs<real> &A, const PassOut &P, cptr<Weights<real>> W,
                                                int wid, real (*ring)[4][LW])
{
    constexpr int q = nodes_of(RT);
    const int lane = threadIdx.x & 63;

    const int nx = A.nx, ny = A.ny, T = A.rows;
    const int nstrip = (nx + 61) / 62, nseg = (ny + T - 1) / T;
    if (wid >= nstrip * nseg) return;  // whole wavefront leaves together
    const int sx = wid % nstrip, sy = wid / nstrip;
    const int x0 = sx * 62, y0 = sy * T;
    const int yend = min(y0 + T, ny);
    const int i = x0 - 1 + lane;
    const bool own_col = lane >= 1 && lane <= 62 && i < nx;
    const bool own = own_col;
    const cptr<real> wtab = weight_table<RT>(W);
    const size_t plane = (size_t)nx * ny;
    const size_t nfx = (size_t)(nx + 1) * ny, nfy = (size_t)nx * (ny + 1);

    // A ring row: columns x0 - 4 .. x0 + 65.  Lane l loads column l of every variable;
    // the six columns left over are loaded by lanes 0..23 together, lane 6 v + k taking
    // column 64 + k of variable v.
    const int sc0 = remap(x0 - 4 + lane, nx, A.bcx);
    const bool has1 = lane < 4 * (LW - 64);
    const int ev = lane / (LW - 64), ec = 64 + lane % (LW - 64);
    const size_t eo = has1 ? ev * plane + remap(x0 - 4 + ec, nx, A.bcx) : sc0;
    const real *__restrict__ Us = A.Us;
    // source row of ring row jr (-4 <= jr <= ny + 4: at most two periods of 4 rows away)
    auto src_row = [&](int jr) {
        if (A.bcy == 0) {
            int r = jr < 0 ? jr + ny : jr;
            r = r >= ny ? r - ny : r;
            return r >= ny ? r - ny : r;
        }
        if (BND && A.bcy == 2) jr = jr < 0 ? -1 - jr : (jr >= ny ? 2 * ny - 1 - jr : jr);
        return jr < 0 ? 0 : (jr >= ny ? ny - 1 : jr);
    };
    struct Row {
        real c[4], e;
    };
    auto load_row = [&](int jr, Row &pf) {
        const size_t rowoff = (size_t)src_row(jr) * nx;
#pragma unroll
        for (int v = 0; v < 4; ++v) pf.c[v] = Us[v * plane + rowoff + sc0];
        pf.e = Us[rowoff + eo];
    };
    // Reflecting walls reverse the x momentum of mirrored columns and the y
    // momentum of mirrored rows; applied here, not at the load, which stays in flight.
    auto store_row = [&](int jr, Row &pf) {
        const int slot = jr & 7;
        // (BND: the build for grids with a reflecting axis or an inflow slit)
        if (BND && A.bcx == 2) {
            const int c0 = x0 - 4 + lane, c1 = x0 - 4 + ec;
            if (c0 < 0 || c0 >= nx) pf.c[1] = -pf.c[1];
            if (ev == 1 && c1 >= nx) pf.e = -pf.e;
        }
        if (BND && A.bcy == 2 && (jr < 0 || jr >= ny)) {
            pf.c[2] = -pf.c[2];
            if (ev == 2) pf.e = -pf.e;
        }
        if (BND && A.slit && (((A.slit & 1) && jr < 0) || ((A.slit & 2) && jr >= ny))) {
            // ghost rows of an inflow slit hold the injected state
            const int c0 = x0 - 4 + lane, c1 = x0 - 4 + ec;
            const int side = jr < 0 ? 0 : 1;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (c0 >= A.si0 && c0 < A.si1) pf.c[v] = A.slitU[side][v];
                if (ev == v && c1 >= A.si0 && c1 < A.si1) pf.e = A.slitU[side][v];
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) ring[slot][v][lane] = pf.c[v];
        if (has1) ring[slot][ev][ec] = pf.e;
    };
    {
        // the first seven rows, all loads in flight together
        Row pf[7];
#pragma unroll
        for (int r = 0; r < 7; ++r) load_row(y0 - 4 + r, pf[r]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < 7; ++r) store_row(y0 - 4 + r, pf[r]);
    }
    wave_lds_sync();

    const real dt = uniform((real)(*A.dt * A.dtf));  // in a scalar register
    const real g = A.gamma;
    real sypP[q][4];   // y+ states of row j-1
    real Gprev[4];     // flux through face j-3/2
    real dFxP[4];      // x-flux difference of row j-1
    bool rsxP = false, rsymP = false;
    unsigned long long tmask = 0ull;  // this lane's lowered cells, bit (row - y0) mod 64
#pragma unroll
    for (int v = 0; v < 4; ++v) { Gprev[v] = real(0); dFxP[v] = real(0); }

    for (int j = y0 - 1; j <= yend; ++j) {
        Row pf;
        load_row(j + 4, pf);  // in flight during this row's arithmetic
        const bool doX = j >= y0 && j < yend;
        const bool first = j == y0 - 1;

        // The x faces, then the y faces: half of the accumulators and states are live at
        // a time.  Each reads the ring through a lane index the compiler takes for a new
        // one, so that the ring's values, and their sums, are read and formed again (8%
        // more instructions) instead of staying in registers in between.
        real dFx[4] = {real(0), real(0), real(0), real(0)};
        bool rsx = false;
        if (doX) {
            real sxm[q][4], sxp[q][4];
            {
                int lx = lane;
                asm volatile("" : "+v"(lx));
                StateAcc<RT, 0, 1, real> acc[4];
                accumulate<RT, ISO>(acc, wtab, [&](int v, int di, int dj) { return ring[(j + dj) & 7][v][lx + 3 + di]; });
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    real m_[q], p_[q];
                    states_of<RT, 0>(acc[v], m_, p_);
#pragma unroll
                    for (int k = 0; k < q; ++k) { sxm[k][v] = m_[k]; sxp[k][v] = p_[k]; }
                }
            }
            real F[4] = {real(0), real(0), real(0), real(0)};
            bool badNb = false;
#pragma unroll
            for (int k = 0; k < q; ++k) {
                real ur[4], f[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) ur[v] = lane_shift<1>(sxm[k][v]);
                bool bl, br;
                riemann<0, HLL>(g, sxp[k], ur, f, bl, br);
                rsx = rsx || bl;
                badNb = badNb || br;
                const real w = node_weight<RT>(A.W, k);
#pragma unroll
                for (int v = 0; v < 4; ++v) F[v] = fma(w, f[v], F[v]);
                hold4(F);  // one node after the other
            }
            // store face i+1/2: lanes of the strip's own cells, plus the domain's left face
            if ((own || (lane == 0 && x0 == 0)) && j < ny) {
                // 32-bit lane offsets from block-uniform bases (fewer live registers)
                const unsigned fi = (unsigned)j * (unsigned)(nx + 1) + (unsigned)(x0 + lane_here());  // face i + 1/2
#pragma unroll
                for (int v = 0; v < 4; ++v) (A.FX + v * nfx)[fi] = F[v];
                A.FXf[fi] = (uint8_t)((rsx ? 1 : 0) | (badNb ? 2 : 0));
            }
            // an inadmissible state on either side of the face troubles both of its
            // cells: this lane's cell takes faces i+1/2 and i-1/2 (the lane below's)
            const bool fbad = rsx || badNb;
            const int badm = lane_shift<-1>((int)fbad);
            rsx = fbad || (badm != 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) dFx[v] = F[v] - lane_shift<-1>(F[v]);
        }

        real sym[q][4], syp[q][4];
        {
            int ly = lane;
            asm volatile("" : "+v"(ly));
            StateAcc<RT, 1, 2, real> acc[4];
            accumulate<RT, ISO>(acc, wtab, [&](int v, int di, int dj) { return ring[(j + dj) & 7][v][ly + 3 + di]; });
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                real m_[q], p_[q];
                states_of<RT, 1>(acc[v], m_, p_);
#pragma unroll
                for (int k = 0; k < q; ++k) { sym[k][v] = m_[k]; syp[k][v] = p_[k]; }
            }
        }

        if (!first) {
            real G[4] = {real(0), real(0), real(0), real(0)};
            bool badLy = false, badRy = false;
            real unp[4] = {real(0), real(0), real(0), real(0)};
            real fh[q / 2 > 0 ? q / 2 : 1][4];  // HLL builds: fluxes of nodes 0 .. q/2-1, paired below
#pragma unroll
            for (int k = 0; k < q; ++k) {
                if (k == q - 1 && A.s != 0 && own && j - 1 >= y0) {
                    // U^n of the cell this row completes, (i, j-1): issued once the
                    // other nodes' states are given up, in flight during this node
                    const unsigned c = (unsigned)(j - 1) * (unsigned)nx + (unsigned)(x0 - 1 + lane_here());
#pragma unroll
                    for (int v = 0; v < 4; ++v) unp[v] = (A.Un + v * plane)[c];
                }
                real f[4];
                bool bl, br;
                riemann<1, HLL>(g, sypP[k], sym[k], f, bl, br);
                badLy = badLy || bl;
                badRy = badRy || br;
                const real w = node_weight<RT>(A.W, k);
                if constexpr (HLL) {
                    // mirror-paired quadrature, (f_k + f_{q-1-k}) w_k: a mirror in x
                    // reverses the nodes of a y face, and the pairs keep the sum exact
                    if (2 * k + 1 < q) {
#pragma unroll
                        for (int v = 0; v < 4; ++v) fh[k < q / 2 ? k : 0][v] = f[v];
                    } else if (2 * k + 1 == q) {
#pragma unroll
                        for (int v = 0; v < 4; ++v) G[v] = fma(w, f[v], G[v]);
                    } else {
                        const int m = q - 1 - k;
#pragma unroll
                        for (int v = 0; v < 4; ++v) G[v] = fma(w, f[v] + fh[m < q / 2 ? m : 0][v], G[v]);
                    }
                } else {
#pragma unroll
                    for (int v = 0; v < 4; ++v) G[v] = fma(w, f[v], G[v]);
                    hold4(G);
                }
            }
            // store face j-1/2 (y index j): the segment's faces above its first row,
            // plus the domain's bottom face
            if (own_col && (j > y0 || y0 == 0)) {
                const unsigned gi = (unsigned)j * (unsigned)nx + (unsigned)(x0 - 1 + lane_here());
#pragma unroll
                for (int v = 0; v < 4; ++v) (A.GY + v * nfy)[gi] = G[v];
                A.GYf[gi] = (uint8_t)((badLy ? 1 : 0) | (badRy ? 2 : 0));
            }
            if (j - 1 >= y0) {
                // cell (i, j-1) is complete
                const int jr = j - 1;
                const int slot = jr & 7;
                real us[4], ust[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    us[v] = ring[slot][v][lane + 3];
                    ust[v] = us[v] - dt * axis_sum(dv(dFxP[v], A.dx), dv(G[v] - Gprev[v], A.dy));
                }
                const bool rs = rsxP || rsymP || badLy || badRy;
                auto nb = [&](int di, int dj, int v) { return ring[(jr + dj) & 7][v][lane + 3 + di]; };
                const bool tr = own && troubled(A, RT, ust, rs, nb);
                if (own) {
                    const unsigned c = (unsigned)jr * (unsigned)nx + (unsigned)(x0 - 1 + lane_here());
#pragma unroll
                    for (int v = 0; v < 4; ++v) (A.Uout + v * plane)[c] = combine(A.s, unp[v], ust[v], A.ca, A.cb);
                    A.order[c] = (uint8_t)(tr ? A.next[RT] : RT);
                }
                // lowered cells are listed once per 64 rows of the march (once per
                // march at the default lengths), not row by row: the wait for the
                // slot an atomic returns would stall the march
                const int rb = (jr - y0) & 63;
                if (tr) tmask |= 1ull << rb;
                if (rb == 63 || jr == yend - 1) {  // the same in every lane
                    const int nt = __popcll(tmask);  // at most 64
                    int b, bt;
                    wave_reserve2(nt | (nt << 16), P.ccount, P.tcount, b, bt);
                    const int row0 = jr - rb;
                    for (unsigned long long m = tmask; m != 0ull; m &= m - 1ull)
                        P.clist[b++] = (row0 + __ffsll((long long)m) - 1) * nx + (x0 - 1 + lane_here());
                    tmask = 0ull;
                }
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) Gprev[v] = G[v];
            rsymP = badLy || badRy;
        }
#pragma unroll
        for (int k = 0; k < q; ++k)
#pragma unroll
            for (int v = 0; v < 4; ++v) sypP[k][v] = syp[k][v];
#pragma unroll
        for (int v = 0; v < 4; ++v) dFxP[v] = dFx[v];
        rsxP = rsx;
        store_row(j + 4, pf);
        wave_lds_sync();
    }
}

// Bound by vector instruction issue: a row of a march is about 2300 vector instructions
// in FP32 and 3400 in FP64 (divisions and square roots are sequences there), against
// 48 and 96 bytes of memory per cell.  So the kernel keeps its instructions to the
// arithmetic and its registers to what lets several marches share a SIMD: 118 vector
// registers in FP32 (four marches), 231 in FP64 (two), nothing spilled.  What that took:
// the weights are read again for every position group (add_group) instead of held in
// scalar registers, which do not hold them all and had every product preceded by a move
// from a spilled one; the row index is scalar; the x faces are finished before the y
// faces begin; sums and node fluxes are formed where they stand (hold4); neighbours'
// states come by lane shifts.  2048^2: 778 -> 502 us a launch in FP64, 301 -> 213 us in
// FP32 (8-row marches), against 5778 -> 3463 and 3152 -> 2354 vector instructions.
template <typename real, int RT, bool ISO, bool HLL, bool BND>
__global__ __launch_bounds__(64, sizeof(real) == 4 ? 4 : 2) void k_first_pass(const StageArgs<real>, const PassOut P)
{
    __shared__ real ring[8][4][LW];
    const StageArgs<real> &A = first_arg<StageArgs<real>>();
    first_pass_wave<real, RT, ISO, HLL, BND>(A, P, &((cptr<StageArgs<real>>)&A)->W, xcd_tile(blockIdx.x, gridDim.x), ring);
}

// ------------------------------------------------------------- cascade pass
// The Riemann solver through a face normal to axis dir (runtime): the momenta are
// swapped into the x-face form and back, so the arithmetic is that of riemann<dir>.
template <bool HLL, typename real>
__device__ __forceinline__ void hllc_rt(real g, int dir, const real (&UL)[4], const real (&UR)[4], real (&F)[4],
                                        bool &badL, bool &badR)
{
    const real L[4] = {UL[0], dir ? UL[2] : UL[1], dir ? UL[1] : UL[2], UL[3]};
    const real Rr[4] = {UR[0], dir ? UR[2] : UR[1], dir ? UR[1] : UR[2], UR[3]};
    real f[4];
    riemann<0, HLL>(g, L, Rr, f, badL, badR);
    F[0] = f[0];
    F[1] = dir ? f[2] : f[1];
    F[2] = dir ? f[1] : f[2];
    F[3] = f[3];
}

// Per-wavefront LDS of the cascade's face work: eight faces of eight lanes, each lane's
// states of its variable and side at up to three nodes, and the nodes' fluxes.
template <typename real>
struct FaceXchg {
    real s[64][3];
    real f[8][3][4];
};

// Copy the compact weight table into LDS (all NT threads of the block, every
// load issued before the first store; a block barrier must follow before it is
// read).
template <int NT, typename real>
__device__ __forceinline__ void load_gtab(const real *gtab, real *wl)
{
    constexpr int per = (kGtabSize + NT - 1) / NT;
    real v[per];
#pragma unroll
    for (int m = 0; m < per; ++m) {
        const int t = (int)threadIdx.x + m * NT;
        v[m] = t < kGtabSize ? gtab[t] : real(0);
    }
#pragma unroll
    for (int m = 0; m < per; ++m) {
        const int t = (int)threadIdx.x + m * NT;
        if (t < kGtabSize) wl[t] = v[m];
    }
}

// The radius-2 diamond, ring by ring.
constexpr int kD13[13][2] = {{0, 0},  {-1, 0}, {1, 0},   {0, -1}, {0, 1},  {-2, 0}, {2, 0},
                             {0, -2}, {0, 2},  {-1, -1}, {1, -1}, {-1, 1}, {1, 1}};

// Columns and row offsets of the cells up to two away from cell (i, j) (unwrapped, at most
// one cell outside the grid), boundary conditions applied.  Returns whether some lane of
// the wavefront (all active) has one of them outside the grid.
template <typename real>
__device__ __forceinline__ bool near_cells(const StageArgs<real> &A, int i, int j, int (&xc)[5], int (&yr)[5])
{
    const int nx = A.nx, ny = A.ny;
    const bool out = __any(((i < 2) | (i >= nx - 2) | (j < 2) | (j >= ny - 2)) != 0) != 0;
    if (!out) {
#pragma unroll
        for (int d = 0; d < 5; ++d) {
            xc[d] = i + d - 2;
            yr[d] = j * nx + (d - 2) * nx;
        }
    } else {
        const AxisMap X(nx, A.bcx), Y(ny, A.bcy);
#pragma unroll
        for (int d = 0; d < 5; ++d) {
            xc[d] = X(i + d - 2);
            yr[d] = Y(j + d - 2) * nx;
        }
    }
    return out;
}

// Cascade pass, part 1: recompute the listed faces at their EDP_1 order (the
// smaller radius of the two cells), eight lanes per face: lane 4 side + v gathers
// variable v around the cell on its side and forms that variable's states at every
// Gauss node; after an LDS transpose lane k solves the Riemann problem of node k, and
// lane v sums variable v of the node fluxes with the Gauss weights (eq. (fvm_F)).  The
// sums and products are those of the first pass, in the same order, with the
// multiplicity of on-axis positions folded into the table weights.
//
// A pass has few faces and waits for each step of this chain in turn, so what counts is
// the length of one lane's instruction stream.  Eight lanes of one side each, the 13
// cells of the diamond loaded once (its positions' mirror images coincide on the axes),
// a transposed face's axes exchanged in the addresses, boundary indices without
// branches and products with the table's zeros left out make it 567 vector instructions
// in FP64 against 1542 with four lanes of both sides and 48 loads each.  With the cells'
// part below, a 160-step run at 512^2 in FP64 went from 306 to 211 ms, a step of the
// 400^2 box with walls from 1.97 to 0.72 ms.
//
// A listed face borders a cell lowered in an earlier evaluation of this stage, so its
// radius is below the top radius: at most 2.  Every lane of the wavefront runs with a
// valid face (lanes past the list repeat an entry and store nothing); wl is the LDS copy
// of the compact weight table.  slot: this lane's place among the per faces of a round.
// pre: when use_pre, its list entry of the first round, loaded by the caller (while the
// count was still unknown; any face id).
template <bool WALLS, bool HLL, typename real>
__device__ __forceinline__ void faces_phase(const StageArgs<real> &A, const real *wl, FaceXchg<real> &X,
                                            const int *flist, unsigned n, unsigned slot, unsigned per, int pre = 0,
                                            bool use_pre = false)
{
    const int nx = A.nx, ny = A.ny;
    const int nfx = (nx + 1) * ny, nfy = nx * (ny + 1);
    const size_t plane = (size_t)nx * ny;
    const int lane = threadIdx.x & 63, l8 = lane & 7, oct = lane >> 3, v = lane & 3, side = (lane >> 2) & 1;
    for (unsigned base = 0; base < n; base += per) {
        const unsigned idx = base + slot;
        if ((unsigned)__builtin_amdgcn_readfirstlane(idx) >= n) break;  // nothing (more) for this wavefront
        const bool valid = idx < n;
        const unsigned f = (unsigned)((use_pre && base == 0) ? pre : flist[valid ? idx : n - 1]);
        const int dir = f >= (unsigned)nfx ? 1 : 0, fo = (int)(dir ? f - (unsigned)nfx : f);
        int i, j;
        split_id(fo, dir ? nx : nx + 1, dir ? A.inv_nx : A.inv_nx1, i, j);
        // this lane's cell: (i, j) on the + side of the face, one step back on the - side
        const int ic = i - (side == 0 && dir == 0 ? 1 : 0), jc = j - (side == 0 && dir == 1 ? 1 : 0);
        int xc[5], yr[5];
        const bool out = near_cells(A, ic, jc, xc, yr);
        const int o = A.order[yr[2] + xc[2]];  // issued ahead of the stencil loads
        // an isotropic y face computes what an x face computes on the transposed
        // grid: position (a, b) is gathered at offset (b, a) and the x table used
        const bool tr = dir == 1 && A.iso;
        const real *U = A.Us + v * plane;
        real q[13];
#pragma unroll
        for (int m = 0; m < 13; ++m) {
            const int a = kD13[m][0] + 2, b = kD13[m][1] + 2;
            q[m] = U[(unsigned)((tr ? yr[a] : xc[a]) + (tr ? xc[b] : yr[b]))];
        }
        if (WALLS) {
            // reflecting walls reverse the normal momentum of mirrored cells; an inflow
            // slit's ghost cells hold the injected state
            // (plain logic on the conditions: no branch per cell)
            if (out) {
                const int fx = (v == 1) & (A.bcx == 2), fy = (v == 2) & (A.bcy == 2);
                real sb[4], st[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    sb[u] = A.slitU[0][u];
                    st[u] = A.slitU[1][u];
                }
                hold4(sb);
                hold4(st);
                const real svb = pick4(v, sb), svt = pick4(v, st);
#pragma unroll
                for (int m = 0; m < 13; ++m) {
                    const int x = ic + (tr ? kD13[m][1] : kD13[m][0]), y = jc + (tr ? kD13[m][0] : kD13[m][1]);
                    const int neg = (fx & ((unsigned)x >= (unsigned)nx)) | (fy & ((unsigned)y >= (unsigned)ny));
                    q[m] *= neg ? real(-1) : real(1);
                    q[m] = in_slit(A, x, y) ? (y < 0 ? svb : svt) : q[m];
                }
            }
        }
        // row_half_mirror: a lane of the other side.  A listed face's radius is at most 2; a
        // lane past the list may hold any face, which is taken at radius 2 as well (its
        // nodes must stay within its own slots of X).
        const int R = min(min(o, dpp<0x141>(o)), 2);
        const real *wt = wl + (R * 2 + (tr ? 0 : dir)) * kGtabPerDir;
        auto w = [&](int p, int e, int c) { return wt[p * (kNPos * 4) + e * 4 + c]; };
        // The parity sums of kQ's positions, the mirror cells of an axis position taken
        // once and doubled (twice at the centre), which is exact.  z: the vanishing sums
        // of the centre (zero, or not a number where the cell is not finite).
        real P[2][4];
        {
            const real ee = (q[0] + q[0]) + (q[0] + q[0]), z = q[0] - q[0];
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                P[p][C_EE] = fma(w(p, 0, C_EE), ee, real(0));
                P[p][C_OE] = P[p][C_EO] = P[p][C_OO] = z;
            }
        }
        auto axis = [&](int e, real plus, real minus, int odd) {
            const real s = plus + minus, d = plus - minus, ee = s + s, od = d + d;
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                P[p][C_EE] = fma(w(p, e, C_EE), ee, P[p][C_EE]);
                P[p][odd] = fma(w(p, e, odd), od, P[p][odd]);
            }
        };
        if (R >= 1) {
            axis(1, q[2], q[1], C_OE);
            axis(2, q[4], q[3], C_EO);
        }
        if (R >= 2) {
            axis(3, q[6], q[5], C_OE);
            axis(4, q[8], q[7], C_EO);
            real d[4];
            parity4(q[12], q[11], q[10], q[9], d);  // (+, +), (-, +), (+, -), (-, -)
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int c = 0; c < 4; ++c) P[p][c] = fma(w(p, 5, c), d[c], P[p][c]);
        }
        // states at the nodes (table order; slot 1 is the centre node of R = 2, a single
        // node has no +- partner): the + face of the lower cell, the - face of the upper
        {
            // odd across / along the face (a transposed y face is in the x-face frame)
            const bool yframe = dir == 1 && !tr;
            const real F0 = yframe ? P[0][C_EO] : P[0][C_OE], N0 = yframe ? P[0][C_OE] : P[0][C_EO];
            const real F1 = yframe ? P[1][C_EO] : P[1][C_OE];
            const real A0 = side ? P[0][C_EE] - F0 : P[0][C_EE] + F0, A1 = side ? P[1][C_EE] - F1 : P[1][C_EE] + F1;
            const real C0 = side ? N0 - P[0][C_OO] : N0 + P[0][C_OO];
            const real sp = A0 + C0, sm = A0 - C0;
            X.s[lane][0] = R <= 0 ? A0 : sp;
            X.s[lane][1] = R == 2 ? A1 : sm;
            X.s[lane][2] = sm;
        }
        wave_lds_sync();
        const int nq = R <= 0 ? 1 : R + 1, k = min(l8, nq - 1);
        real fk[4];
        bool bl, br;
        {
            real UL[4], UR[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                UL[u] = X.s[oct * 8 + u][k];
                UR[u] = X.s[oct * 8 + 4 + u][k];
            }
            hllc_rt<HLL>(A.gamma, dir, UL, UR, fk, bl, br);
        }
        // the lanes past the last node repeat it: no need to leave them out
        const unsigned ml = (unsigned)(__ballot(bl) >> (oct * 8)) & 0xffu, mr = (unsigned)(__ballot(br) >> (oct * 8)) & 0xffu;
        if (l8 < nq) {
#pragma unroll
            for (int u = 0; u < 4; ++u) X.f[oct][l8][u] = fk[u];
        }
        wave_lds_sync();
        if (valid && side == 0) {
            const real *qw = wl + kGtabNodeOff + R * 2;
            real F;
            if constexpr (HLL) {
                // mirror-paired quadrature (see the first pass's y faces)
                if (R <= 0) F = fma(qw[0], X.f[oct][0][v], real(0));
                else if (R == 1) F = fma(qw[0], X.f[oct][1][v] + X.f[oct][0][v], real(0));
                else F = fma(qw[0], X.f[oct][2][v] + X.f[oct][0][v], fma(qw[1], X.f[oct][1][v], real(0)));
            } else {
                F = fma(qw[0], X.f[oct][0][v], real(0));
                if (R >= 1) F = fma(R >= 2 ? qw[1] : qw[0], X.f[oct][1][v], F);
                if (R >= 2) F = fma(qw[0], X.f[oct][2][v], F);
            }
            const uint8_t fl = (uint8_t)((ml ? 1 : 0) | (mr ? 2 : 0));
            if (dir == 0) {
                A.FX[(size_t)v * nfx + fo] = F;
                if (v == 0) A.FXf[fo] = fl;
            } else {
                A.GY[(size_t)v * nfy + fo] = F;
                if (v == 0) A.GYf[fo] = fl;
            }
        }
        wave_lds_sync();  // the next round overwrites X
    }
}

// Cascade pass, part 2: re-evaluate the listed cells from the stored fluxes,
// re-detect, lower the troubled ones and claim the faces and cells of the next
// pass.  Detection reads no other cell's order, so lowering in place is safe.
//
// Four lanes per cell, for the same reason as the eight per face: lane w updates
// variable w, holds the face neighbour w (west, east, south, north) with its pressure
// and normal velocity, and claims face w and neighbour w; what the others need passes
// by quad moves.  The candidate, the bounds and the verdict are the same in all four.
// Every lane of the wavefront runs with a valid cell (lanes past the list repeat an
// entry, store nothing and claim nothing), so the quad moves see no idle lane.
//
// cell_load gathers what does not depend on this pass's fluxes (the stage input
// around the cell, U^n and its order); cell_finish reads the fluxes and flags,
// forms the candidate, detects, writes the result and lowers.  The tail issues
// cell_load while other wavefronts still recompute the faces.
template <typename real>
struct CellIn {
    int c, i, j, o;
    real us, un;   // U_s and U^n of the cell, variable w
    real nb[4];    // face neighbour w
    real r8[8];    // densities of the outer ring of the radius-2 diamond (kD13[5..12])
};

template <bool WALLS, typename real>
__device__ __forceinline__ void cell_load(const StageArgs<real> &A, int c, CellIn<real> &X)
{
    const int nx = A.nx, ny = A.ny, w = threadIdx.x & 3;
    const size_t plane = (size_t)nx * ny;
    X.c = c;
    split_id(c, nx, A.inv_nx, X.i, X.j);
    int xc[5], yr[5];
    const bool out = near_cells(A, X.i, X.j, xc, yr);
    const int di = w == 0 ? -1 : (w == 1 ? 1 : 0), dj = w == 2 ? -1 : (w == 3 ? 1 : 0);
    const unsigned nbi = (unsigned)((w == 2 ? yr[1] : (w == 3 ? yr[3] : yr[2])) + (w == 0 ? xc[1] : (w == 1 ? xc[3] : xc[2])));
    X.us = (A.Us + w * plane)[c];
#pragma unroll
    for (int u = 0; u < 4; ++u) X.nb[u] = (A.Us + u * plane)[nbi];
#pragma unroll
    for (int m = 0; m < 8; ++m) X.r8[m] = A.Us[(unsigned)(yr[kD13[5 + m][1] + 2] + xc[kD13[5 + m][0] + 2])];
    X.un = A.s == 0 ? real(0) : (A.Un + w * plane)[c];
    X.o = A.order[c];
    // reflecting walls reverse the normal momentum of a mirrored face neighbour;
    // an inflow slit's ghost cells hold the injected state
    if (WALLS) {
        if (out) {
            const int x = X.i + di, y = X.j + dj;
            const int nx1 = (A.bcx == 2) & ((unsigned)x >= (unsigned)nx), ny1 = (A.bcy == 2) & ((unsigned)y >= (unsigned)ny);
            X.nb[1] *= nx1 ? real(-1) : real(1);
            X.nb[2] *= ny1 ? real(-1) : real(1);
            if (A.slit) {
                real sb[4], st[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    sb[u] = A.slitU[0][u];
                    st[u] = A.slitU[1][u];
                }
                hold4(sb);
                hold4(st);
                const bool s = in_slit(A, x, y);
#pragma unroll
                for (int u = 0; u < 4; ++u) X.nb[u] = s ? (y < 0 ? sb[u] : st[u]) : X.nb[u];
#pragma unroll
                for (int m = 0; m < 8; ++m) {
                    const int xm = X.i + kD13[5 + m][0], ym = X.j + kD13[5 + m][1];
                    X.r8[m] = in_slit(A, xm, ym) ? (ym < 0 ? sb[0] : st[0]) : X.r8[m];
                }
            }
        }
    }
}

// Returns whether the cell is troubled (it has then been lowered; the same in its four
// lanes).  valid: this lane's cell is one of the list (else nothing is stored).
template <typename real>
__device__ __forceinline__ bool cell_finish(const StageArgs<real> &A, const CellIn<real> &X, real dt, bool valid)
{
    const int nx = A.nx, ny = A.ny, w = threadIdx.x & 3;
    const size_t plane = (size_t)nx * ny;
    const size_t nfx = (size_t)(nx + 1) * ny, nfy = (size_t)nx * (ny + 1);
    const unsigned fxm = (unsigned)(X.j * (nx + 1) + X.i), gym = (unsigned)(X.j * nx + X.i);  // faces i-1/2, j-1/2
    const real *FX = A.FX + w * nfx, *GY = A.GY + w * nfy;
    const real f0 = FX[fxm], f1 = FX[fxm + 1], f2 = GY[gym], f3 = GY[gym + (unsigned)nx];
    int fl = (w < 2 ? A.FXf : A.GYf)[w == 0 ? fxm : (w == 1 ? fxm + 1 : (w == 2 ? gym : gym + (unsigned)nx))];
    const real mine = X.us - dt * axis_sum(dv(f1 - f0, A.dx), dv(f3 - f2, A.dy));
    if (valid) (A.Uout + w * plane)[X.c] = combine(A.s, X.un, mine, A.ca, A.cb);
    // an inadmissible state on either side of any of the cell's faces
    fl |= dpp<0xb1>(fl);  // quad_perm:[1,0,3,2]
    fl |= dpp<0x4e>(fl);  // quad_perm:[2,3,0,1]
    const real rho = quad<0>(mine), mx = quad<1>(mine), my = quad<2>(mine), E = quad<3>(mine);
    const real g = A.gamma;
    // Detection (Steps 4-10), as troubled()
    const real p = pressure(g, rho, mx, my, E);
    const bool bad = !(finite(rho) && finite(p))             // Step 4: CAD
                     || ((A.flags & 8u) && fl != 0)          // CAD on the Riemann states
                     || !(rho > real(0) && p > real(0));     // Step 5: PAD
    // DMP bounds over the cell and its face neighbours
    const real rc = quad<0>(X.us), rW = quad<0>(X.nb[0]), rE = quad<1>(X.nb[0]), rS = quad<2>(X.nb[0]), rN = quad<3>(X.nb[0]);
    real lo = rc, hi = rc;
    lo = vmin(lo, rW); hi = vmax(hi, rW);
    lo = vmin(lo, rE); hi = vmax(hi, rE);
    lo = vmin(lo, rS); hi = vmax(hi, rS);
    lo = vmin(lo, rN); hi = vmax(hi, rN);
    bool open = X.o != 0 && !bad && !(lo <= rho && rho <= hi);                 // Step 10; Step 8: DMP
    open = open && !((A.flags & 2u) && (hi - lo) < A.plat_thr);                // Step 7: plateau
    if ((A.flags & 1u) && __any(open)) {                                       // Step 6: CSD
        const real pn = pressure(g, X.nb[0], X.nb[1], X.nb[2], X.nb[3]);
        const real un = dv(w < 2 ? X.nb[1] : X.nb[2], X.nb[0]);
        // the x terms in lanes 0 and 1, the y terms in lanes 2 and 3
        const real plo = dpp<0xa0>(pn), phi = dpp<0xf5>(pn);  // quad_perm:[0,0,2,2], [1,1,3,3]
        const real ulo = dpp<0xa0>(un), uhi = dpp<0xf5>(un);
        const real td = real(2) * (w < 2 ? A.dx : A.dy);
        const real du = dv(uhi - ulo, td), dp = dv(fabs(phi - plo), td * vmin(phi, plo));
        const real divV = quad<0>(du) + quad<2>(du), gradp = quad<0>(dp) + quad<2>(dp);
        open = open && !(divV >= -A.sigma_v && gradp <= A.sigma_p);
    }
    if ((A.flags & 4u) && __any(open)) {                                       // Step 9: u2
        // lanes 0 and 2 take the curvatures in x, lanes 1 and 3 those in y
        const bool y = (w & 1) != 0;
        const real w0 = y ? A.W.curv[1][0] : A.W.curv[0][0], wa = y ? A.W.curv[1][1] : A.W.curv[0][1];
        const real wt = y ? A.W.curv[1][2] : A.W.curv[0][2];
        const real rho5[5] = {rc, rW, rE, rS, rN};
        // sums of the x pair and the y pair around the cell and its face neighbours
        const real sx[5] = {rW + rE, X.r8[0] + rc, rc + X.r8[1], X.r8[4] + X.r8[5], X.r8[6] + X.r8[7]};
        const real sy[5] = {rS + rN, X.r8[4] + X.r8[6], X.r8[5] + X.r8[7], X.r8[2] + rc, rc + X.r8[3]};
        real cmin = real(0), cmax = real(0);
#pragma unroll
        for (int m = 0; m < 5; ++m) {
            real kap = w0 * rho5[m];
            kap = fma(wa, y ? sy[m] : sx[m], kap);
            kap = fma(wt, y ? sx[m] : sy[m], kap);
            cmin = m == 0 ? kap : vmin(cmin, kap);
            cmax = m == 0 ? kap : vmax(cmax, kap);
        }
        const bool prod = cmin * cmax > -A.delta;
        const bool a = prod && vmax(fabs(cmax), fabs(cmin)) < A.delta;
        const bool b = prod && fabs(cmin) >= real(0.5) * fabs(cmax);
        const int ok = (a || b) ? 1 : 0;
        open = open && !(quad<0>(ok) != 0 && quad<1>(ok) != 0);
    }
    const bool tr = valid && X.o != 0 && (bad || open);
    if (tr && w == 0) A.order[X.c] = (uint8_t)next_radius(A.next[0], A.next[1], A.next[2], A.next[3], X.o);
    return tr;
}

// Claims after lowering cell (i, j) (act: this quad's cell was lowered): its four faces
// (and, on periodic axes, the duplicate copy of a boundary face) are listed for
// recomputation in the next pass, and the cell with its four face neighbours for
// re-evaluation; *P.tcount counts the lowered cells (null: not counted).  A stamp per face and per
// cell keeps each list duplicate-free.  Lane w of the quad claims face w (x faces i,
// i + 1 of row j; y faces j, j + 1 of column i) and face neighbour w, lane 0 the cell
// itself, lanes 1 and 2 the duplicates: three atomics a lane in flight together, list
// slots from ballots and one reservation per wavefront and list.  Must be reached by all
// 64 lanes of the wavefront together.
template <typename real>
__device__ __forceinline__ void claim_after_lowering(const StageArgs<real> &A, const PassOut &P, int i, int j,
                                                     bool act)
{
    const unsigned long long any = __ballot(act);
    if (any == 0ull) return;
    const int nx = A.nx, ny = A.ny, lane = threadIdx.x & 63, w = lane & 3;
    const unsigned nfx = (unsigned)((nx + 1) * ny);
    const unsigned fx = (unsigned)(j * (nx + 1) + i), gy = nfx + (unsigned)(j * nx + i);
    const unsigned fid = w == 0 ? fx : (w == 1 ? fx + 1 : (w == 2 ? gy : gy + (unsigned)nx));
    const int ii = i + (w == 0 ? -1 : (w == 1 ? 1 : 0)), jj = j + (w == 2 ? -1 : (w == 3 ? 1 : 0));
    const bool cok = (A.bcx == 0 || (ii >= 0 && ii < nx)) && (A.bcy == 0 || (jj >= 0 && jj < ny));
    // (on a non-periodic axis only in-domain indices get here: no mirror needed)
    const int cid = wrap(jj, ny, A.bcy) * nx + wrap(ii, nx, A.bcx);
    // lane 1: the copy of x face 0 / face nx; lane 2: of y face 0 / face ny
    const bool dup = (w == 1 && A.bcx == 0 && (i == 0 || i == nx - 1)) || (w == 2 && A.bcy == 0 && (j == 0 || j == ny - 1));
    const unsigned did = w == 1 ? (unsigned)(j * (nx + 1) + (i == 0 ? nx : 0)) : nfx + (unsigned)((j == 0 ? ny * nx : 0) + i);
    unsigned a0 = P.stamp, a1 = P.stamp, a2 = P.stamp;
    if (act) {
        a0 = atomicMax(&A.fstamp[fid], P.stamp);
        if (cok) a1 = atomicMax(&A.cstamp[cid], P.stamp);
        if (w == 0) a2 = atomicMax(&A.cstamp[j * nx + i], P.stamp);
        else if (dup) a2 = atomicMax(&A.fstamp[did], P.stamp);
    }
    const bool m0 = a0 < P.stamp, m1 = a1 < P.stamp, m2 = a2 < P.stamp;  // newly claimed here
    const unsigned long long bf0 = __ballot(m0), bc1 = __ballot(m1), bf2 = __ballot(m2 && w != 0), bc2 = __ballot(m2 && w == 0);
    const int nf0 = __popcll(bf0), nc1 = __popcll(bc1);
    unsigned fb = 0;
    int cb = 0;
    if (lane == 0) {
        fb = (unsigned)atomicAdd(P.fcount, nf0 + __popcll(bf2));
        cb = atomicAdd(P.ccount, nc1 + __popcll(bc2));
        if (P.tcount) atomicAdd(P.tcount, __popcll(any) >> 2);
    }
    fb = __builtin_amdgcn_readfirstlane(fb);
    cb = __builtin_amdgcn_readfirstlane(cb);
    if (m0) P.flist[fb + (unsigned)below(bf0)] = (int)fid;
    if (m1) P.clist[cb + below(bc1)] = cid;
    if (m2 && w == 0) P.clist[cb + nc1 + below(bc2)] = j * nx + i;
    if (m2 && w != 0) P.flist[fb + (unsigned)(nf0 + below(bf2))] = (int)did;
}

template <bool WALLS, typename real>
__device__ __forceinline__ void cells_phase(const StageArgs<real> &A, const int *clist, int n, int slot, int per,
                                            const PassOut &P, real dt, int pre = 0, bool use_pre = false)
{
    for (int base = 0; base < n; base += per) {
        const int idx = base + slot;
        if (__builtin_amdgcn_readfirstlane(idx) >= n) break;  // nothing (more) for this wavefront
        const bool valid = idx < n;
        CellIn<real> X;
        cell_load<WALLS>(A, (use_pre && base == 0) ? pre : clist[valid ? idx : n - 1], X);
        const bool tr = cell_finish(A, X, dt, valid);
        claim_after_lowering(A, P, X.i, X.j, tr);
    }
}

// The claims of the cells the first pass lowered (listed in low, count *nlow):
// the same claims, stamps and lists as if they had been made in the pass.
template <typename real>
__global__ __launch_bounds__(256) void k_claims_first(const StageArgs<real> A, const PassOut P, const int *low,
                                                      const int *nlow)
{
    const int n = *nlow;
    PassOut Q = P;
    Q.stamp = *A.stamp0;
    Q.tcount = nullptr;  // the first pass has counted them
    const unsigned stride = gridDim.x * blockDim.x;
    for (unsigned r = 0; quad_item(r, stride, 0) < (unsigned)n; ++r) {
        const int t = (int)quad_item(r, stride, blockIdx.x * blockDim.x + threadIdx.x);
        const bool act = t < n;
        int i = 0, j = 0;
        if (act) split_id(low[t], A.nx, A.inv_nx, i, j);
        claim_after_lowering(A, Q, i, j, act);
    }
}

// Outputs of cascade pass k.
__device__ __forceinline__ PassOut pass_out(const Cascade &C, int k, unsigned stamp0)
{
    PassOut P;
    P.flist = C.flist[(k + 1) & 1];
    P.fcount = &C.ctl->nface[k + 1];
    P.clist = C.clist[(k + 1) & 1];
    P.ccount = &C.ctl->ncell[k + 1];
    P.tcount = &C.ctl->ntroub[k];
    P.stamp = stamp0 + (unsigned)k;
    return P;
}

// Does multi-block pass k run?  Not when it has nothing to do, nor when the
// previous evaluation left few troubled cells (the tail takes over from k).
__device__ __forceinline__ bool pass_runs(const Cascade &C, int k)
{
    return C.ctl->ncell[k] > 0 && C.ctl->ntroub[k - 1] > C.tail_thr;
}

template <typename real, bool WALLS, bool HLL>
__global__ __launch_bounds__(256) void k_faces(const StageArgs<real>, const Cascade C, int k)
{
    const StageArgs<real> &A = first_arg<StageArgs<real>>();
    __shared__ real wl[kGtabSize];
    __shared__ FaceXchg<real> xch[4];
    const unsigned cap = faces_of(A.nx, A.ny);
    const unsigned t0 = blockIdx.x * blockDim.x + threadIdx.x;
    // issued together, before the counts are known: this thread's first list
    // entry (in bounds; used only if the pass runs and covers it) and the weights
    const unsigned i0 = t0 >> 3;
    const int pre = C.flist[k & 1][i0 < cap ? i0 : cap - 1];
    load_gtab<256>(A.gtab, wl);
    if (!pass_runs(C, k)) {
        if (blockIdx.x == 0 && threadIdx.x == 0 && C.ctl->ncell[k] > 0) C.ctl->tail_k0 = k;
        return;
    }
    unsigned n = (unsigned)C.ctl->nface[k];
    n = n < cap ? n : cap;  // a list holds each face at most once
    if (n <= blockIdx.x * 32) return;  // no face for this block
    __syncthreads();
    faces_phase<WALLS, HLL>(A, wl, xch[threadIdx.x >> 6], C.flist[k & 1], n, i0, gridDim.x * 32, pre, true);
}

template <typename real, bool WALLS>
__global__ __launch_bounds__(256) void k_cells(const StageArgs<real>, const Cascade C, int k)
{
    const StageArgs<real> &A = first_arg<StageArgs<real>>();
    const int cap = A.nx * A.ny;
    const int t0 = blockIdx.x * blockDim.x + threadIdx.x;
    // this quad's first list entry, issued before the counts are known (in bounds; a
    // list only ever holds cells of the grid)
    const int i0 = t0 >> 2;
    const int pre = C.clist[k & 1][i0 < cap ? i0 : cap - 1];
    const real dt = (real)(*A.dt * A.dtf);
    if (!pass_runs(C, k)) return;
    int n = C.ctl->ncell[k];
    n = n < cap ? n : cap;  // a list holds each cell at most once
    if (n <= (int)(blockIdx.x * 64)) return;
    cells_phase<WALLS>(A, C.clist[k & 1], n, i0, gridDim.x * 64, pass_out(C, k, C.ctl->stamp0), dt, pre, true);
}

// The tail of a long cascade (few troubled cells per pass) in one workgroup:
// passes run back to back with block barriers, from tail_k0 (or kdef when the
// multi-block passes did not hand over), until a pass has no cell to re-evaluate,
// kend is reached, or the previous evaluation left more than back_thr troubled
// cells (hand back to the multi-block passes).  The counts of the running passes
// stay in LDS and are copied to the control block as each pass completes.  kbeg 0 (then
// kdef is 1): the claims of the first pass's lowered cells are not made yet; the tail makes
// them, unless they are more than back_thr (hand back at once).
// Threads of the tail workgroup: as many as its registers allow (four wavefronts per SIMD
// in FP32, three in FP64).
template <typename real>
constexpr int tail_threads()
{
    return sizeof(real) == 8 ? 768 : 1024;
}

// LDS of the single-workgroup cascade.
template <typename real>
struct TailShared {
    real wl[kGtabSize];
    FaceXchg<real> xch[tail_threads<real>() / 64];
    int cnt[2][3];  // [pass parity][faces, cells, troubled cells of the previous evaluation]
    int kfirst;
};

template <bool WALLS, bool HLL, typename real>
__device__ __forceinline__ void tail_body(const StageArgs<real> &A, const Cascade &C, int kbeg, int kdef, int kend,
                                          TailShared<real> &S)
{
    const unsigned capf = faces_of(A.nx, A.ny);
    const int capc = A.nx * A.ny;
    Ctl *ctl = C.ctl;
    const unsigned stamp0 = ctl->stamp0;
    const real dtr = (real)(*A.dt * A.dtf);  // read once, not after each pass's barrier
    load_gtab<tail_threads<real>()>(A.gtab, S.wl);
    const int handed = ctl->tail_k0;
    int k0 = handed > 0 ? handed : kdef;
    const bool claims = kbeg == 0;
    if (handed <= 0 && !claims && kbeg < kdef) {
        // no hand-over: the cascade either ended inside the batch kbeg..kdef-1 (at
        // the first pass with no cell) or continues at kdef
        if (threadIdx.x == 0) S.kfirst = kdef;
        __syncthreads();
        for (int kk = kbeg + (int)threadIdx.x; kk < kdef; kk += blockDim.x)
            if (ctl->ncell[kk] <= 0) atomicMin(&S.kfirst, kk);
        __syncthreads();
        k0 = S.kfirst;
    }
    if (threadIdx.x == 0) {
        S.cnt[k0 & 1][0] = ctl->nface[k0];
        S.cnt[k0 & 1][1] = ctl->ncell[k0];
        S.cnt[k0 & 1][2] = ctl->ntroub[k0 - 1];
    }
    int k = k0;
    bool back = false;
    if (claims) {
        // a kernel for a few claims costs more than they do (64^2 FP64 step 201 -> 190 us,
        // RK4 at 200^2 218 -> 211 us)
        const int nlow = __builtin_amdgcn_readfirstlane(ctl->nlow);
        if (nlow > C.back_thr) {
            back = true;
        } else {
            __syncthreads();  // the counts are set
            PassOut P = pass_out(C, 0, stamp0);
            P.fcount = &S.cnt[k0 & 1][0];
            P.ccount = &S.cnt[k0 & 1][1];
            P.tcount = nullptr;  // the first pass has counted them
            for (int m = (int)threadIdx.x >> 2; __builtin_amdgcn_readfirstlane(m) < nlow; m += tail_threads<real>() / 4) {
                int i = 0, j = 0;
                if (m < nlow) split_id(C.clist[0][m], A.nx, A.inv_nx, i, j);
                claim_after_lowering(A, P, i, j, m < nlow);
            }
        }
    }
    for (; !back && k < kend; ++k) {
        __syncthreads();  // the previous pass's lists, counts and fluxes are complete
        // the same value in every lane: held in scalar registers, so the branches
        // below (some around block barriers) are scalar
        unsigned nf = (unsigned)__builtin_amdgcn_readfirstlane(S.cnt[k & 1][0]);
        int nc = __builtin_amdgcn_readfirstlane(S.cnt[k & 1][1]);
        const int nt = __builtin_amdgcn_readfirstlane(S.cnt[k & 1][2]);
        if (threadIdx.x == 0 && (claims || k > k0)) {
            ctl->nface[k] = (int)nf;
            ctl->ncell[k] = nc;
            ctl->ntroub[k - 1] = nt;
        }
        nc = nc < capc ? nc : capc;
        nf = nf < capf ? nf : capf;
        if (nc <= 0) break;  // same values in every thread: the block leaves together
        if (nt > C.back_thr) {
            back = true;
            break;
        }
        if (threadIdx.x == 0) S.cnt[(k + 1) & 1][0] = S.cnt[(k + 1) & 1][1] = S.cnt[(k + 1) & 1][2] = 0;
        PassOut P = pass_out(C, k, stamp0);
        P.fcount = &S.cnt[(k + 1) & 1][0];
        P.ccount = &S.cnt[(k + 1) & 1][1];
        P.tcount = &S.cnt[(k + 1) & 1][2];
        const int fw = (int)groups_of(nf, 8), cw = (int)groups_of(nc, 16);  // wavefronts of faces, of cells
        const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);  // uniform per wavefront
        if (fw + cw <= tail_threads<real>() / 64) {
            // one round each, on separate wavefronts: the cell wavefronts gather
            // their inputs while the face wavefronts recompute the fluxes
            const int c0 = tail_threads<real>() / 64 - cw;  // first cell wavefront
            const bool cellwave = wv >= c0;
            const int idx = ((int)threadIdx.x - 64 * c0) >> 2;
            CellIn<real> X;
            if (cellwave) cell_load<WALLS>(A, C.clist[k & 1][idx < nc ? idx : nc - 1], X);
            else if (wv < fw)
                faces_phase<WALLS, HLL>(A, S.wl, S.xch[wv], C.flist[k & 1], nf, threadIdx.x >> 3, 8 * fw);
            __syncthreads();
            if (cellwave) claim_after_lowering(A, P, X.i, X.j, cell_finish(A, X, dtr, idx < nc));
        } else {
            faces_phase<WALLS, HLL>(A, S.wl, S.xch[wv], C.flist[k & 1], nf, threadIdx.x >> 3, tail_threads<real>() / 8);
            __syncthreads();
            cells_phase<WALLS>(A, C.clist[k & 1], nc, threadIdx.x >> 2, tail_threads<real>() / 4, P, dtr);
        }
    }
    if (k >= kend) {
        __syncthreads();
        if (threadIdx.x == 0) {
            ctl->nface[k] = S.cnt[k & 1][0];
            ctl->ncell[k] = S.cnt[k & 1][1];
            ctl->ntroub[k - 1] = S.cnt[k & 1][2];
        }
    }
    if (threadIdx.x == 0) {
        if (C.report) {
            // straight into pinned host memory: a copy after the kernel takes 4 us and a gap
            C.report[0] = k;
            C.report[1] = back ? 1 : 0;
            C.report[2] = k0;
        }
        ctl->tail_end = k;
        ctl->tail_back = back ? 1 : 0;
        ctl->tail_start = k0;
        if (back) ctl->tail_k0 = 0;  // the next multi-block batch starts afresh
    }
}

template <typename real, bool WALLS, bool HLL>
__global__ __launch_bounds__((tail_threads<real>())) void k_tail(const StageArgs<real>, const Cascade C, int kbeg, int kdef,
                                                       int kend)
{
    const StageArgs<real> &A = first_arg<StageArgs<real>>();
    __shared__ TailShared<real> S;
    tail_body<WALLS, HLL>(A, C, kbeg, kdef, kend, S);
}

// -------------------------------------------------------- small kernels
__global__ void k_reset(Ctl *ctl, int nzero, unsigned stamp0)
{
    for (int k = threadIdx.x; k < nzero && k < kMaxPasses + 2; k += blockDim.x) {
        ctl->nface[k] = 0;
        ctl->ncell[k] = 0;
        ctl->ntroub[k] = 0;
    }
    if (threadIdx.x == 0) {
        ctl->tail_end = 0;
        ctl->tail_k0 = 0;
        ctl->tail_back = 0;
        ctl->stamp0 = stamp0;
        ctl->nlow = 0;
    }
}

// Histogram of the final cascade level of every cell (for statistics only).
__global__ __launch_bounds__(256) void k_level_hist(const uint8_t *order, size_t ncell, const LevIdx levidx,
                                                    unsigned long long *levcnt)
{
    __shared__ unsigned int h[4];
    if (threadIdx.x < 4) h[threadIdx.x] = 0;
    __syncthreads();
    unsigned int loc[4] = {0, 0, 0, 0};
    for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < ncell; k += (size_t)gridDim.x * blockDim.x) {
        const int r = order[k] & 3;
        loc[0] += r == 0;
        loc[1] += r == 1;
        loc[2] += r == 2;
        loc[3] += r == 3;
    }
    for (int r = 0; r < 4; ++r)
        if (loc[r]) atomicAdd(&h[r], loc[r]);
    __syncthreads();
    if (threadIdx.x < 4 && h[threadIdx.x]) atomicAdd(&levcnt[levidx.v[threadIdx.x]], (unsigned long long)h[threadIdx.x]);
}

__global__ void k_zero_levcnt(Ctl *ctl)
{
    if (threadIdx.x < 4) ctl->levcnt[threadIdx.x] = 0ull;
}

// Instrumentation: add this stage's final-order counts and MOOD iterations
// (1 + cascade passes that re-evaluated cells) to the accumulators.
__global__ void k_stats_accum(Ctl *ctl, int npass, int reset)
{
    __shared__ unsigned long long cnt;
    if (threadIdx.x == 0) cnt = 0ull;
    __syncthreads();
    if (reset) {
        if (threadIdx.x < 4) ctl->acc_lev[threadIdx.x] = 0ull;
        if (threadIdx.x == 0) {
            ctl->acc_iters = 0ull;
            ctl->acc_stages = 0ull;
        }
        return;
    }
    unsigned long long loc = 0;
    for (int k = 1 + threadIdx.x; k <= npass && k < kMaxPasses + 2; k += blockDim.x) loc += ctl->ncell[k] > 0;
    if (loc) atomicAdd(&cnt, loc);
    __syncthreads();
    if (threadIdx.x < 4) ctl->acc_lev[threadIdx.x] += ctl->levcnt[threadIdx.x];
    if (threadIdx.x == 0) {
        ctl->acc_iters += 1ull + cnt;
        ctl->acc_stages += 1ull;
    }
}

// max over cells of (|u_d| + c) / Delta_d in FP64, as the bit pattern of a
// non-negative double (which orders like the integer).
template <typename real>
__device__ __forceinline__ void dt_reduce_body(const real *U, size_t ncell, double gamma, double dx, double dy,
                                               unsigned long long *lam_bits, size_t first, size_t stride,
                                               double *red)
{
    double lam = 0.0;
    // four cells per round, their 16 loads issued before the arithmetic (the
    // maximum does not depend on the order)
    constexpr int kU = 4;
    for (size_t k0 = first; k0 < ncell; k0 += kU * stride) {
        double q[kU][4];
#pragma unroll
        for (int m = 0; m < kU; ++m) {
            const size_t k = k0 + (size_t)m * stride;
            const size_t kk = k < ncell ? k : first;  // in bounds; the cell is skipped below
#pragma unroll
            for (int v = 0; v < 4; ++v) q[m][v] = U[(size_t)v * ncell + kk];
        }
#pragma unroll
        for (int m = 0; m < kU; ++m) {
            if (k0 + (size_t)m * stride >= ncell) continue;
            const double r = q[m][0], mx = q[m][1], my = q[m][2], E = q[m][3];
            const double p = (gamma - 1.0) * (E - 0.5 * (mx * mx + my * my) / r);
            if (!(r > 0.0 && p > 0.0 && __builtin_isfinite(r) && __builtin_isfinite(p))) continue;
            const double cs = sqrt(gamma * p / r);
            const double lx = (fabs(mx / r) + cs) / dx;
            const double ly = (fabs(my / r) + cs) / dy;
            const double l = lx > ly ? lx : ly;
            lam = l > lam ? l : lam;
        }
    }
    red[threadIdx.x] = lam;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] = red[threadIdx.x] > red[threadIdx.x + s] ? red[threadIdx.x] : red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0 && red[0] > 0.0) {
        // the maximum only grows (the bit patterns of positive doubles order as
        // the values): a block whose value does not exceed the one already stored
        // skips its atomic, so the blocks do not queue on the one address
        const unsigned long long b = (unsigned long long)__double_as_longlong(red[0]);
        if (b > __hip_atomic_load(lam_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(lam_bits, b);
    }
}

template <typename real>
__global__ __launch_bounds__(256) void k_dt_reduce(const real *U, size_t ncell, double gamma, double dx,
                                                   double dy, unsigned long long *lam_bits)
{
    __shared__ double red[256];
    dt_reduce_body(U, ncell, gamma, dx, dy, lam_bits, (size_t)blockIdx.x * blockDim.x + threadIdx.x,
                   (size_t)gridDim.x * blockDim.x, red);
}

// lam0: a lower bound of the largest wave speed over cell size (an inflow slit's
// state), 0 if none.
__global__ void k_dt_finalize(Ctl *ctl, double cfl, double lam0)
{
    const double lam = __longlong_as_double((long long)ctl->lam_bits);
    ctl->dt = cfl / (lam > lam0 ? lam : lam0);
}

__global__ void k_dt_set(Ctl *ctl, double dt, int clear_lambda)
{
    if (clear_lambda) ctl->lam_bits = 0ull;
    else ctl->dt = dt;
}

// out = w0 x0 + w1 x1 + w2 x2 + w3 x3, evaluated left to right, element by element.
template <typename real>
__global__ __launch_bounds__(256) void k_lincomb4(real *out, const real *x0, const real *x1, const real *x2,
                                                  const real *x3, real w0, real w1, real w2, real w3, size_t n)
{
    for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (size_t)gridDim.x * blockDim.x)
        out[k] = ((w0 * x0[k] + w1 * x1[k]) + w2 * x2[k]) + w3 * x3[k];
}

// Compensated totals: per-block double-double partial sums in a fixed order.
__device__ __forceinline__ void two_sum(double a, double b, double &s, double &e)
{
    s = a + b;
    const double bb = s - a;
    e = (a - (s - bb)) + (b - bb);
}

__device__ __forceinline__ void dd_add(double &hi, double &lo, double x)
{
    double s, e;
    two_sum(hi, x, s, e);
    e += lo;
    two_sum(s, e, hi, lo);
}

template <typename real>
__global__ __launch_bounds__(256) void k_totals_partial(const real *U, size_t ncell, double *partial)
{
    __shared__ double sh[256], sl[256];
    const int v = blockIdx.y;
    double hi = 0.0, lo = 0.0;
    for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < ncell; k += (size_t)gridDim.x * blockDim.x)
        dd_add(hi, lo, (double)U[v * ncell + k]);
    sh[threadIdx.x] = hi;
    sl[threadIdx.x] = lo;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            double h = sh[threadIdx.x], l = sl[threadIdx.x];
            dd_add(h, l, sh[threadIdx.x + s]);
            dd_add(h, l, sl[threadIdx.x + s]);
            sh[threadIdx.x] = h;
            sl[threadIdx.x] = l;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        partial[(v * gridDim.x + blockIdx.x) * 2] = sh[0];
        partial[(v * gridDim.x + blockIdx.x) * 2 + 1] = sl[0];
    }
}

__global__ void k_totals_final(const double *partial, int nblk, double area, double *out)
{
    const int v = threadIdx.x;
    if (v >= 4) return;
    double hi = 0.0, lo = 0.0;
    for (int b = 0; b < nblk; ++b) {
        dd_add(hi, lo, partial[(v * nblk + b) * 2]);
        dd_add(hi, lo, partial[(v * nblk + b) * 2 + 1]);
    }
    out[v] = (hi + lo) * area;
}

// ------------------------------------------------------------- launchers
// ------------------------------------------------------------ batched ensemble
// Many independent problems advance together: one first-pass launch over all
// their strips, one single-workgroup cascade per problem in one launch, and the
// per-problem dt in three small launches.  The per-problem arguments live in
// device tables written once; they are read through the constant address space
// (scalar loads: the tables do not change while the kernels run).
// Generic reference to entry p of a device table, loaded as constant memory.
template <typename T>
__device__ __forceinline__ const T &table_entry(const T *tab, int p)
{
    return *(const T *)(((cptr<T>)tab) + p);
}

template <typename Prefix>
__device__ __forceinline__ int find_problem(Prefix prefix, int n, int b)
{
    int lo = 0, hi = n;  // prefix[lo] <= b < prefix[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (prefix[mid] <= b) lo = mid;
        else hi = mid;
    }
    return lo;
}

template <typename real, int RT, bool ISO, bool HLL, bool BND>
__global__ __launch_bounds__(64, sizeof(real) == 4 ? 4 : 2) void k_first_pass_batch(const BatchTabs<real> B)
{
    __shared__ real ring[8][4][LW];
    cptr<int> blk = (cptr<int>)B.blk;
    const int p = find_problem(blk, B.nprob, blockIdx.x);
    const StageArgs<real> &A = table_entry(B.args, p);
    const Cascade &C = table_entry(B.casc, p);
    PassOut Q = table_entry(B.pout, p);
    // lowered cells are listed in clist[0]; k_claims_first_batch makes their claims
    Q.clist = C.clist[0];
    Q.ccount = &C.ctl->nlow;
    first_pass_wave<real, RT, ISO, HLL, BND>(A, Q, &(((cptr<StageArgs<real>>)B.args) + p)->W, blockIdx.x - blk[p], ring);
}

// Multi-block cascade passes of a batch.  Before each pass, k_batch_plan (or k_faces_batch) sizes
// every problem's share of the pass (0 when it has no work, or when its previous
// evaluation left at most tail_thr troubled cells, which then leaves the rest of
// its cascade to its tail workgroup) and lays the shares end to end: plan[p] is
// the first work block of problem p, in units of 32 faces and, at plan + nprob + 1, of
// 64 cells (256 threads each).  The pass kernels have a fixed grid whose
// blocks stride over these work blocks, so the whole batch's faces and cells of a
// pass are spread over the GPU however they fall among the problems.  Pass 0 is
// the claims of the cells the first passes lowered (64 cells per block).
constexpr int kBatchPasses = 12;
constexpr int kBatchFaceGrid = 1024, kBatchCellGrid = 2048;

// Work blocks of faces (df) and of cells (dc) of problem p in pass k >= 1; a problem that
// leaves the rest of its cascade to its tail is told so (mark: by this thread).
template <typename real>
__device__ __forceinline__ void batch_share(const BatchTabs<real> &B, int p, int k, bool mark, int &df, int &dc)
{
    const StageArgs<real> &A = table_entry(B.args, p);
    const Cascade &C = table_entry(B.casc, p);
    const unsigned capf = faces_of(A.nx, A.ny), nf = (unsigned)C.ctl->nface[k];
    const int capc = A.nx * A.ny, nc = C.ctl->ncell[k], nt = C.ctl->ntroub[k - 1];  // loaded together
    const bool runs = nc > 0 && nt > C.tail_thr;  // pass_runs
    df = runs ? (int)groups_of(min(nf, capf), 32) : 0;
    dc = runs ? (min(nc, capc) + 63) / 64 : 0;
    if (mark && !runs && nc > 0) C.ctl->tail_k0 = k;  // the tail takes over from this pass
}

template <typename real>
__global__ __launch_bounds__(1024) void k_batch_plan(const BatchTabs<real> B, int k, int *plan)
{
    __shared__ int sf[1024], sc[1024];
    __shared__ int carry[2];
    if (threadIdx.x == 0) carry[0] = carry[1] = 0;
    for (int base = 0; base < B.nprob; base += blockDim.x) {
        const int p = base + (int)threadIdx.x;
        int df = 0, dc = 0;
        if (p < B.nprob) {
            if (k == 0) df = (table_entry(B.casc, p).ctl->nlow + 63) / 64;
            else batch_share(B, p, k, true, df, dc);
        }
        sf[threadIdx.x] = df;
        sc[threadIdx.x] = dc;
        __syncthreads();
        // inclusive scan (Hillis-Steele) of both demands
        for (int off = 1; off < (int)blockDim.x; off <<= 1) {
            const int tf = threadIdx.x >= (unsigned)off ? sf[threadIdx.x - off] : 0;
            const int tc = threadIdx.x >= (unsigned)off ? sc[threadIdx.x - off] : 0;
            __syncthreads();
            sf[threadIdx.x] += tf;
            sc[threadIdx.x] += tc;
            __syncthreads();
        }
        if (p < B.nprob) {
            plan[p] = carry[0] + sf[threadIdx.x] - df;
            plan[B.nprob + 1 + p] = carry[1] + sc[threadIdx.x] - dc;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            carry[0] += sf[blockDim.x - 1];
            carry[1] += sc[blockDim.x - 1];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        plan[B.nprob] = carry[0];
        plan[2 * B.nprob + 1] = carry[1];
    }
}

// The claims of the cells each problem's first pass lowered.
template <typename real>
__global__ __launch_bounds__(256) void k_claims_first_batch(const BatchTabs<real> B, const int *plan)
{
    cptr<int> pl = (cptr<int>)plan;
    const int total = pl[B.nprob];
    for (int w = blockIdx.x; w < total; w += gridDim.x) {
        const int p = find_problem(pl, B.nprob, w);
        const StageArgs<real> &A = table_entry(B.args, p);
        const Cascade &C = table_entry(B.casc, p);
        PassOut P = table_entry(B.pout, p);
        P.stamp = *A.stamp0;
        P.tcount = nullptr;  // the first pass has counted them
        const int t = (int)quad_item(w - pl[p], 256, threadIdx.x);
        const bool act = t < C.ctl->nlow;
        int i = 0, j = 0;
        if (act) split_id(C.clist[0][t], A.nx, A.inv_nx, i, j);
        claim_after_lowering(A, P, i, j, act);
    }
}

// PLAN: at most 256 problems; every block then lays out the shares itself, one problem a
// thread, and block 0 writes the cells' for k_cells_batch (a launch of k_batch_plan before
// each pass took 4.8 us and a gap: 12 FP32 problems of 64^2 to 320^2, 7.07 -> 6.26 ms for six
// steps).  The line is the block's 256 threads, and it still pays there: a step of problems
// of 64^2 with the kernel before each pass against this, FP32 (FP64), 12 problems 657 532 us
// (792 666), 64 892 761 (1069 943), 128 1090 984 (1427 1328), 256 1521 1475 (2148 2113);
// 256 of 200^2 4486 4438 (7891 7852).
template <typename real, bool WALLS, bool HLL, bool PLAN>
__global__ __launch_bounds__(256) void k_faces_batch(const BatchTabs<real> B, int k, int *plan)
{
    __shared__ real wl[kGtabSize];
    __shared__ FaceXchg<real> xch[4];
    __shared__ int first[PLAN ? 257 : 1], part[2][4];
    cptr<int> pl = (cptr<int>)plan;
    if constexpr (PLAN) {
        const int p = threadIdx.x, lane = p & 63, wv = p >> 6;
        int df = 0, dc = 0;
        if (p < B.nprob) batch_share(B, p, k, blockIdx.x == 0, df, dc);
        int f = df, c = dc;  // sums up to this problem
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int tf = __shfl_up(f, d), tc = __shfl_up(c, d);
            f += lane >= d ? tf : 0;
            c += lane >= d ? tc : 0;
        }
        if (lane == 63) {
            part[0][wv] = f;
            part[1][wv] = c;
        }
        __syncthreads();
        for (int w = 0; w < wv; ++w) {
            f += part[0][w];
            c += part[1][w];
        }
        first[p + 1] = f;  // beyond the last problem: the total
        if (p == 0) first[0] = 0;
        if (blockIdx.x == 0 && p < B.nprob) {
            if (p == 0) plan[B.nprob + 1] = 0;
            plan[B.nprob + 2 + p] = c;
        }
        __syncthreads();
    }
    const int total = PLAN ? __builtin_amdgcn_readfirstlane(first[PLAN ? B.nprob : 0]) : pl[B.nprob];
    int loaded = -1;  // problem whose weights wl holds
    for (int w = blockIdx.x; w < total; w += gridDim.x) {
        const int p = PLAN ? __builtin_amdgcn_readfirstlane(find_problem((const int *)first, B.nprob, w)) : find_problem(pl, B.nprob, w);
        const StageArgs<real> &A = table_entry(B.args, p);
        const Cascade &C = table_entry(B.casc, p);
        if (p != loaded) {
            __syncthreads();  // the previous work block's readers of wl are done
            load_gtab<256>(A.gtab, wl);
            __syncthreads();
            loaded = p;
        }
        const unsigned n = min((unsigned)C.ctl->nface[k], faces_of(A.nx, A.ny));
        faces_phase<WALLS, HLL>(A, wl, xch[threadIdx.x >> 6], C.flist[k & 1], n,
                                (unsigned)(w - (PLAN ? first[PLAN ? p : 0] : pl[p])) * 32 + (threadIdx.x >> 3), n);
    }
}

template <typename real, bool WALLS>
__global__ __launch_bounds__(256) void k_cells_batch(const BatchTabs<real> B, int k, const int *plan)
{
    cptr<int> pl = (cptr<int>)(plan + B.nprob + 1);
    const int total = pl[B.nprob];
    for (int w = blockIdx.x; w < total; w += gridDim.x) {
        const int p = find_problem(pl, B.nprob, w);
        const StageArgs<real> &A = table_entry(B.args, p);
        const Cascade &C = table_entry(B.casc, p);
        const int n = min(C.ctl->ncell[k], A.nx * A.ny);
        cells_phase<WALLS>(A, C.clist[k & 1], n, (w - pl[p]) * 64 + ((int)threadIdx.x >> 2), n,
                           pass_out(C, k, C.ctl->stamp0), (real)(*A.dt * A.dtf));
    }
}

// Problem p = blockIdx.x runs the rest of its cascade in one workgroup, from the
// pass the multi-block passes left to it (no hand-back).
template <typename real, bool WALLS, bool HLL>
__global__ __launch_bounds__((tail_threads<real>())) void k_tail_batch(const BatchTabs<real> B)
{
    __shared__ TailShared<real> S;
    const int p = blockIdx.x;
    const StageArgs<real> &A = table_entry(B.args, p);
    const Cascade &C = table_entry(B.casc, p);
    tail_body<WALLS, HLL>(A, C, 1, kBatchPasses + 1, kMaxPasses, S);
}

// Stage start of every problem: counts of evaluation 0 and pass 1, tail state,
// and a fresh claim stamp range (kMaxPasses + 2 stamps per stage).
__global__ void k_reset_batch(const Cascade *casc, int nprob)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= nprob) return;
    Ctl *ctl = casc[p].ctl;
    // the counts the first pass and the multi-block passes add to
    for (int k = 0; k <= kBatchPasses + 1; ++k) {
        ctl->nface[k] = 0;
        ctl->ncell[k] = 0;
        ctl->ntroub[k] = 0;
    }
    ctl->tail_end = 0;
    ctl->tail_k0 = 0;
    ctl->tail_back = 0;
    ctl->nlow = 0;
    ctl->stamp0 += (unsigned)kMaxPasses + 2;
}

// The stamp range restarts after the stamp arrays were cleared.
__global__ void k_stamp_restart_batch(const Cascade *casc, int nprob)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < nprob) casc[p].ctl->stamp0 = 0u;
}

__global__ void k_dt_begin_batch(const Cascade *casc, int nprob)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < nprob) casc[p].ctl->lam_bits = 0ull;
}

// Blocks dblk[p] .. dblk[p+1]-1 reduce problem p's U^n (the stage-0 input).
template <typename real>
__global__ __launch_bounds__(256) void k_dt_reduce_batch(const BatchTabs<real> B)
{
    __shared__ double red[256];
    cptr<int> dblk = (cptr<int>)B.dblk;
    const int p = find_problem(dblk, B.nprob, blockIdx.x);
    const StageArgs<real> &A = table_entry(B.args, p);
    const Cascade &C = table_entry(B.casc, p);
    const int lb = blockIdx.x - dblk[p], nb = dblk[p + 1] - dblk[p];
    dt_reduce_body(A.Us, (size_t)A.nx * A.ny, A.gamma64, A.dx64, A.dy64, &C.ctl->lam_bits,
                   (size_t)lb * blockDim.x + threadIdx.x, (size_t)nb * blockDim.x, red);
}

__global__ void k_dt_end_batch(const Cascade *casc, int nprob, double cfl)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < nprob) {
        Ctl *ctl = casc[p].ctl;
        ctl->dt = cfl / __longlong_as_double((long long)ctl->lam_bits);
    }
}

// Per problem: evaluations of the last stage (0 if its cascade hit the pass
// limit) and dt.
__global__ void k_batch_status(const Cascade *casc, int nprob, int *iters, double *dts)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < nprob) {
        const Ctl *ctl = casc[p].ctl;
        iters[p] = ctl->tail_end >= kMaxPasses ? 0 : ctl->tail_end;
        dts[p] = ctl->dt;
    }
}

// The cascade of a batch stage after its first pass: the claims of the lowered
// cells, kBatchPasses multi-block passes, then one workgroup per problem.
template <typename real, bool WALLS, bool HLL>
static hipError_t launch_batch_cascade(const BatchTabs<real> &B, hipStream_t st)
{
    hipLaunchKernelGGL(k_batch_plan<real>, dim3(1), dim3(1024), 0, st, B, 0, B.plan);
    hipLaunchKernelGGL(k_claims_first_batch<real>, dim3(kBatchFaceGrid), dim3(256), 0, st, B, (const int *)B.plan);
    for (int k = 1; k <= kBatchPasses; ++k) {
        if (B.nprob <= 256) {
            hipLaunchKernelGGL((k_faces_batch<real, WALLS, HLL, true>), dim3(kBatchFaceGrid), dim3(256), 0, st, B, k,
                               B.plan);
        } else {
            hipLaunchKernelGGL(k_batch_plan<real>, dim3(1), dim3(1024), 0, st, B, k, B.plan);
            hipLaunchKernelGGL((k_faces_batch<real, WALLS, HLL, false>), dim3(kBatchFaceGrid), dim3(256), 0, st, B, k,
                               B.plan);
        }
        hipLaunchKernelGGL((k_cells_batch<real, WALLS>), dim3(kBatchCellGrid), dim3(256), 0, st, B, k,
                           (const int *)B.plan);
    }
    hipLaunchKernelGGL((k_tail_batch<real, WALLS, HLL>), dim3(B.nprob), dim3(tail_threads<real>()), 0, st, B);
    return hipGetLastError();
}

// BW: the first-pass build with the boundary handling (some problem has walls).
template <typename real, bool BW>
static hipError_t launch_batch_stage_bw(const BatchTabs<real> &B, int top, int nfp_blocks, const Cascade *casc,
                                        hipStream_t st, bool tail = true)
{
    const int nb = (B.nprob + 255) / 256;
    hipLaunchKernelGGL(k_reset_batch, dim3(nb), dim3(256), 0, st, casc, B.nprob);
    const dim3 g(nfp_blocks), t(64);
    if (B.solver == 1) {
        switch (top * 2 + (B.iso ? 1 : 0)) {
        case 7: hipLaunchKernelGGL((k_first_pass_batch<real, 3, true, true, BW>), g, t, 0, st, B); break;
        case 6: hipLaunchKernelGGL((k_first_pass_batch<real, 3, false, true, BW>), g, t, 0, st, B); break;
        case 5: hipLaunchKernelGGL((k_first_pass_batch<real, 2, true, true, BW>), g, t, 0, st, B); break;
        case 4: hipLaunchKernelGGL((k_first_pass_batch<real, 2, false, true, BW>), g, t, 0, st, B); break;
        case 3: hipLaunchKernelGGL((k_first_pass_batch<real, 1, true, true, BW>), g, t, 0, st, B); break;
        case 2: hipLaunchKernelGGL((k_first_pass_batch<real, 1, false, true, BW>), g, t, 0, st, B); break;
        default: return hipErrorInvalidValue;
        }
        if (!tail) return hipGetLastError();
        return B.walls ? launch_batch_cascade<real, true, true>(B, st) : launch_batch_cascade<real, false, true>(B, st);
    }
    switch (top * 2 + (B.iso ? 1 : 0)) {
    case 7: hipLaunchKernelGGL((k_first_pass_batch<real, 3, true, false, BW>), g, t, 0, st, B); break;
    case 6: hipLaunchKernelGGL((k_first_pass_batch<real, 3, false, false, BW>), g, t, 0, st, B); break;
    case 5: hipLaunchKernelGGL((k_first_pass_batch<real, 2, true, false, BW>), g, t, 0, st, B); break;
    case 4: hipLaunchKernelGGL((k_first_pass_batch<real, 2, false, false, BW>), g, t, 0, st, B); break;
    case 3: hipLaunchKernelGGL((k_first_pass_batch<real, 1, true, false, BW>), g, t, 0, st, B); break;
    case 2: hipLaunchKernelGGL((k_first_pass_batch<real, 1, false, false, BW>), g, t, 0, st, B); break;
    default: return hipErrorInvalidValue;
    }
    if (!tail) return hipGetLastError();
    return B.walls ? launch_batch_cascade<real, true, false>(B, st) : launch_batch_cascade<real, false, false>(B, st);
}

template <typename real>
hipError_t launch_batch_stage(const BatchTabs<real> &B, int top, int nfp_blocks, const Cascade *casc,
                              hipStream_t st)
{
    return B.walls ? launch_batch_stage_bw<real, true>(B, top, nfp_blocks, casc, st)
                   : launch_batch_stage_bw<real, false>(B, top, nfp_blocks, casc, st);
}

// The reset and the first pass of a batch stage without its cascade (timing).
template <typename real>
hipError_t launch_batch_first_pass(const BatchTabs<real> &B, int top, int nfp_blocks, const Cascade *casc,
                                   hipStream_t st)
{
    return B.walls ? launch_batch_stage_bw<real, true>(B, top, nfp_blocks, casc, st, false)
                   : launch_batch_stage_bw<real, false>(B, top, nfp_blocks, casc, st, false);
}

template <typename real>
hipError_t launch_batch_dt(const BatchTabs<real> &B, int ndt_blocks, const Cascade *casc, double cfl, hipStream_t st)
{
    const int nb = (B.nprob + 255) / 256;
    hipLaunchKernelGGL(k_dt_begin_batch, dim3(nb), dim3(256), 0, st, casc, B.nprob);
    hipLaunchKernelGGL(k_dt_reduce_batch<real>, dim3(ndt_blocks), dim3(256), 0, st, B);
    hipLaunchKernelGGL(k_dt_end_batch, dim3(nb), dim3(256), 0, st, casc, B.nprob, cfl);
    return hipGetLastError();
}

hipError_t launch_batch_status(const Cascade *casc, int nprob, int *iters, double *dts, hipStream_t st)
{
    hipLaunchKernelGGL(k_batch_status, dim3((nprob + 255) / 256), dim3(256), 0, st, casc, nprob, iters, dts);
    return hipGetLastError();
}

hipError_t launch_batch_stamp_restart(const Cascade *casc, int nprob, hipStream_t st)
{
    hipLaunchKernelGGL(k_stamp_restart_batch, dim3((nprob + 255) / 256), dim3(256), 0, st, casc, nprob);
    return hipGetLastError();
}

template <typename real, int RT>
static hipError_t launch_first_pass_rt(const StageArgs<real> &A, const PassOut &P, hipStream_t st)
{
    const dim3 g(first_pass_waves(A.nx, A.ny, A.rows)), t(64);
    const int bnd = (A.bcx == 2 || A.bcy == 2 || A.slit != 0) ? 4 : 0;
    switch (bnd + (A.solver == 1 ? 2 : 0) + (A.iso ? 1 : 0)) {
    case 0: hipLaunchKernelGGL((k_first_pass<real, RT, false, false, false>), g, t, 0, st, A, P); break;
    case 1: hipLaunchKernelGGL((k_first_pass<real, RT, true, false, false>), g, t, 0, st, A, P); break;
    case 2: hipLaunchKernelGGL((k_first_pass<real, RT, false, true, false>), g, t, 0, st, A, P); break;
    case 3: hipLaunchKernelGGL((k_first_pass<real, RT, true, true, false>), g, t, 0, st, A, P); break;
    case 4: hipLaunchKernelGGL((k_first_pass<real, RT, false, false, true>), g, t, 0, st, A, P); break;
    case 5: hipLaunchKernelGGL((k_first_pass<real, RT, true, false, true>), g, t, 0, st, A, P); break;
    case 6: hipLaunchKernelGGL((k_first_pass<real, RT, false, true, true>), g, t, 0, st, A, P); break;
    default: hipLaunchKernelGGL((k_first_pass<real, RT, true, true, true>), g, t, 0, st, A, P); break;
    }
    return hipGetLastError();
}

// First pass, then the claims of the cells it lowered (listed in C.clist[0],
// which pass 1 only writes after reading its own list C.clist[1]); `mid`, if
// given, is recorded between the two.
template <typename real>
hipError_t launch_first_claims(const StageArgs<real> &A, const PassOut &P, const Cascade &C, hipStream_t st)
{
    hipLaunchKernelGGL(k_claims_first<real>, dim3(256), dim3(256), 0, st, A, P, C.clist[0], &C.ctl->nlow);
    return hipGetLastError();
}

template <typename real>
hipError_t launch_first_pass(const StageArgs<real> &A, const PassOut &P, const Cascade &C, hipEvent_t mid, bool claims,
                             hipStream_t st)
{
    PassOut Q = P;
    Q.clist = C.clist[0];
    Q.ccount = &C.ctl->nlow;
    hipError_t e;
    switch (A.top) {
    case 3: e = launch_first_pass_rt<real, 3>(A, Q, st); break;
    case 2: e = launch_first_pass_rt<real, 2>(A, Q, st); break;
    case 1: e = launch_first_pass_rt<real, 1>(A, Q, st); break;
    default: return hipErrorInvalidValue;
    }
    if (e == hipSuccess && mid) e = hipEventRecord(mid, st);
    return e == hipSuccess && claims ? launch_first_claims<real>(A, P, C, st) : e;
}

template <typename real>
hipError_t launch_cascade_pass(const StageArgs<real> &A, const Cascade &C, int k, int nblocks, hipStream_t st)
{
    const bool walls = A.bcx == 2 || A.bcy == 2 || A.slit != 0;
    if (walls && A.solver == 1)
        hipLaunchKernelGGL((k_faces<real, true, true>), dim3(nblocks), dim3(256), 0, st, A, C, k);
    else if (walls)
        hipLaunchKernelGGL((k_faces<real, true, false>), dim3(nblocks), dim3(256), 0, st, A, C, k);
    else if (A.solver == 1)
        hipLaunchKernelGGL((k_faces<real, false, true>), dim3(nblocks), dim3(256), 0, st, A, C, k);
    else
        hipLaunchKernelGGL((k_faces<real, false, false>), dim3(nblocks), dim3(256), 0, st, A, C, k);
    if (walls)
        hipLaunchKernelGGL((k_cells<real, true>), dim3(nblocks), dim3(256), 0, st, A, C, k);
    else
        hipLaunchKernelGGL((k_cells<real, false>), dim3(nblocks), dim3(256), 0, st, A, C, k);
    return hipGetLastError();
}

template <typename real>
hipError_t launch_cascade_tail(const StageArgs<real> &A, const Cascade &C, int kbeg, int kdef, int kend,
                               hipStream_t st)
{
    const bool walls = A.bcx == 2 || A.bcy == 2 || A.slit != 0;
    if (walls && A.solver == 1)
        hipLaunchKernelGGL((k_tail<real, true, true>), dim3(1), dim3(tail_threads<real>()), 0, st, A, C, kbeg, kdef, kend);
    else if (walls)
        hipLaunchKernelGGL((k_tail<real, true, false>), dim3(1), dim3(tail_threads<real>()), 0, st, A, C, kbeg, kdef, kend);
    else if (A.solver == 1)
        hipLaunchKernelGGL((k_tail<real, false, true>), dim3(1), dim3(tail_threads<real>()), 0, st, A, C, kbeg, kdef, kend);
    else
        hipLaunchKernelGGL((k_tail<real, false, false>), dim3(1), dim3(tail_threads<real>()), 0, st, A, C, kbeg, kdef, kend);
    return hipGetLastError();
}

hipError_t launch_reset(Ctl *ctl, int nzero, unsigned stamp0, hipStream_t st)
{
    hipLaunchKernelGGL(k_reset, dim3(1), dim3(256), 0, st, ctl, nzero, stamp0);
    return hipGetLastError();
}

hipError_t launch_level_hist(const uint8_t *order, size_t ncell, const LevIdx &levidx, Ctl *ctl, hipStream_t st)
{
    hipLaunchKernelGGL(k_zero_levcnt, dim3(1), dim3(64), 0, st, ctl);
    size_t nblk = (ncell + 255) / 256;
    if (nblk > 1024) nblk = 1024;
    hipLaunchKernelGGL(k_level_hist, dim3((unsigned)nblk), dim3(256), 0, st, order, ncell, levidx, ctl->levcnt);
    return hipGetLastError();
}

template <typename real>
hipError_t launch_lincomb4(real *out, const real *x0, const real *x1, const real *x2, const real *x3, double w0,
                           double w1, double w2, double w3, size_t n, hipStream_t st)
{
    size_t nb = (n + 255) / 256;
    if (nb > 8192) nb = 8192;
    hipLaunchKernelGGL(k_lincomb4<real>, dim3((unsigned)nb), dim3(256), 0, st, out, x0, x1, x2, x3, (real)w0,
                       (real)w1, (real)w2, (real)w3, n);
    return hipGetLastError();
}

template <typename real>
hipError_t launch_dt(const real *U, size_t ncell, double gamma, double dx, double dy, double cfl, double lam0, Ctl *ctl,
                     hipStream_t st)
{
    hipLaunchKernelGGL(k_dt_set, dim3(1), dim3(1), 0, st, ctl, 0.0, 1);
    size_t nblk = (ncell + 255) / 256;
    if (nblk > 4096) nblk = 4096;
    hipLaunchKernelGGL(k_dt_reduce<real>, dim3((unsigned)nblk), dim3(256), 0, st, U, ncell, gamma, dx, dy,
                       &ctl->lam_bits);
    hipLaunchKernelGGL(k_dt_finalize, dim3(1), dim3(1), 0, st, ctl, cfl, lam0);
    return hipGetLastError();
}

hipError_t launch_stats(Ctl *ctl, int npass, int reset, hipStream_t st)
{
    hipLaunchKernelGGL(k_stats_accum, dim3(1), dim3(256), 0, st, ctl, npass, reset);
    return hipGetLastError();
}

hipError_t launch_set_dt(Ctl *ctl, double dt, hipStream_t st)
{
    hipLaunchKernelGGL(k_dt_set, dim3(1), dim3(1), 0, st, ctl, dt, 0);
    return hipGetLastError();
}

template <typename real>
hipError_t launch_totals(const real *U, size_t ncell, double area, double *partial, int nblk, double *out,
                         hipStream_t st)
{
    hipLaunchKernelGGL(k_totals_partial<real>, dim3(nblk, 4), dim3(256), 0, st, U, ncell, partial);
    hipLaunchKernelGGL(k_totals_final, dim3(1), dim3(64), 0, st, partial, nblk, area, out);
    return hipGetLastError();
}

template hipError_t launch_first_pass<float>(const StageArgs<float> &, const PassOut &, const Cascade &, hipEvent_t, bool,
                                              hipStream_t);
template hipError_t launch_first_pass<double>(const StageArgs<double> &, const PassOut &, const Cascade &, hipEvent_t, bool,
                                               hipStream_t);
template hipError_t launch_first_claims<float>(const StageArgs<float> &, const PassOut &, const Cascade &, hipStream_t);
template hipError_t launch_first_claims<double>(const StageArgs<double> &, const PassOut &, const Cascade &, hipStream_t);
template hipError_t launch_cascade_pass<float>(const StageArgs<float> &, const Cascade &, int, int, hipStream_t);
template hipError_t launch_cascade_pass<double>(const StageArgs<double> &, const Cascade &, int, int, hipStream_t);
template hipError_t launch_cascade_tail<float>(const StageArgs<float> &, const Cascade &, int, int, int, hipStream_t);
template hipError_t launch_cascade_tail<double>(const StageArgs<double> &, const Cascade &, int, int, int,
                                                hipStream_t);
template hipError_t launch_lincomb4<float>(float *, const float *, const float *, const float *, const float *,
                                           double, double, double, double, size_t, hipStream_t);
template hipError_t launch_lincomb4<double>(double *, const double *, const double *, const double *,
                                            const double *, double, double, double, double, size_t, hipStream_t);
template hipError_t launch_dt<float>(const float *, size_t, double, double, double, double, double, Ctl *, hipStream_t);
template hipError_t launch_dt<double>(const double *, size_t, double, double, double, double, double, Ctl *, hipStream_t);
template hipError_t launch_totals<float>(const float *, size_t, double, double *, int, double *, hipStream_t);
template hipError_t launch_totals<double>(const double *, size_t, double, double *, int, double *, hipStream_t);

template hipError_t launch_batch_stage<float>(const BatchTabs<float> &, int, int, const Cascade *, hipStream_t);
template hipError_t launch_batch_first_pass<float>(const BatchTabs<float> &, int, int, const Cascade *, hipStream_t);
template hipError_t launch_batch_first_pass<double>(const BatchTabs<double> &, int, int, const Cascade *, hipStream_t);
template hipError_t launch_batch_stage<double>(const BatchTabs<double> &, int, int, const Cascade *, hipStream_t);
template hipError_t launch_batch_dt<float>(const BatchTabs<float> &, int, const Cascade *, double, hipStream_t);
template hipError_t launch_batch_dt<double>(const BatchTabs<double> &, int, const Cascade *, double, hipStream_t);

}  // namespace gpm
