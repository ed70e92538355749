// swe_nest.hpp -- gfx950 kernels of hierarchical (nested) grids.
//
// Method: arXiv 1705.00614, Sec. 2.2 (a hierarchy of grids in which the
// small-scale flow of a zoomed-in area feeds back into the large-scale grid)
// and Sec. 5 (a 50 m global grid with a 12.5 m local grid).  The paper does
// not spell out the coupling; the one implemented here is coarse-first
// subcycling with conservative flux matching.  Per coarse step:
//
//   coarse   one ordinary step of the coarse grid with time step tau_c; the
//            step adds tau_c * flux of the faces bounding every covered box
//            into its taps
//   r times  k_frame fills the frame of every patch (the FRAME cells round
//            its interior, one more than the reach of one step) from the
//            covering coarse cell, linear in time between the coarse layers
//            n and n+1 (depth and discharge interpolated; fine depth
//            H_f = max(0, H_c + b_c - b_fine) and discharge H_f Q_c / H_c
//            where the coarse cell is wet, else dry); then one ordinary
//            step of every patch with tau_c / r,
//            adding tau_f * flux of its interior boundary faces into its taps
//   feedback k_feedback: each covered coarse cell takes the mean of its
//            r x r fine cells; each uncovered cell next to a covered box
//            takes (coarse tap - mean of the r fine taps of the same coarse
//            face) / h_c through that face, with the final update's clamp,
//            ledger and dry rule, the momentum part weighted by the cell's
//            depth after it (NEST_MOMENTUM_DEPTH); then k_nest_close
//            gathers the CFL speed of the changed cells, puts the tiles
//            round the covered boxes on the coarse tile list and clears the
//            taps, its last workgroup setting the steps as below
//   tau      (k_nest_tau without feedback, which also clears the taps)
//            tau_c = min(CFL step of the
//            coarse speeds, r * CFL step of every patch after its last
//            substep), tau_f = tau_c / r, and the coarse hydrograph volume of
//            the next step.
//
// All of it is device work on one stream (capturable in a graph); the host
// only launches.
#pragma once

#include <algorithm>
#include <vector>

#include "swe_step.hpp"

namespace swe {

constexpr int NEST_FRAME = 5;   // frame width in fine cells
// patches of a nest at most (the time-step rule reads one per lane of a wave)
constexpr int NEST_MAX_PATCHES = 64;
// ring cells shallower than this [m] after the reflux take its mass but not
// its momentum, twice as deep all of it, linear between (a film moving with
// the patch's flow would set the nest's CFL step through the friction term
// of U_p)
constexpr double NEST_MOMENTUM_DEPTH = 0.05;

template <typename real>
struct NestPatch {
    int ci0, cj0, cw, ch;          // covered coarse box
    int nxe, nye;                  // extended fine grid (interior + frame)
    int ftap, ctap;                // offsets of the patch's and the coarse box's taps
    real* Hf[2]; real* Qxf[2]; real* Qyf[2];
    const real* bf;
    Ctrl* ctrl;
    const double* mass;            // the patch's per-tile FP64 depth sums
    int ntx, tx, ty;               // its tile columns and tile shape
};

template <typename real>
struct NestArgs {
    const NestPatch<real>* P;
    int np, r, nx, ny;             // patches, refinement, coarse grid
    int nring;                     // ring cells (all patches)
    real* Hc[2]; real* Qxc[2]; real* Qyc[2];
    const real* bc;
    real* tap;
    const int* ring_cell;          // coarse cell of each ring cell
    const int* ring_off;           // CSR offsets into ring_face (nring + 1)
    const int* ring_face;          // per face: patch, side (0 W, 1 E, 2 S, 3 N), index along the side
    double* ring_ledger;           // clamp volume per ring cell (accumulated)
    real eps, ih;                  // dry threshold, 1 / h_c
    double h2;                     // h_c^2
    double hold;                   // held coarse step length (0: the CFL rule)
};

// Shares of a launch over the grids of a nest with these tile counts, and the
// grids' order in it (nest_shares): about GROUPS groups of NSEG workgroups,
// twice what is resident at once, in proportion to the tiles, but no more than
// one workgroup per tile and no fewer than LEAST groups while there are tiles
// for them (a workgroup strides over further tiles; one without a tile holds
// its place for a read of the control block only).  Us per two-way coarse step
// in FP32, r = 2 but where said.  A 2048^2 lake with 16 patches of one tile:
// as many workgroups for each grid 780, so 171 (a launch per grid 446).  A
// 1024^2 lake with nine patches of 160^2, r = 4: 64 groups 707, 128 592, 256
// 569; two patches of 4096 tiles, about 700 of them listed, r = 4: 212, 211,
// 212.  A dry 2048^2 grid with nine wet patches of 25 tiles: at least 1 group
// 100, 8 79, 32 79.
constexpr int NEST_GROUPS = 128, NEST_LEAST = 8;
inline GridShares nest_shares(const std::vector<int>& tiles, std::vector<int>& order) {
    const int n = (int)tiles.size();
    long long sum = 0;
    for (int t : tiles) sum += t;
    std::vector<int> m(n);
    for (int k = 0; k < n; ++k)
        m[k] = std::min((tiles[k] + NSEG - 1) / NSEG,
                        std::max(NEST_LEAST, (int)((long long)NEST_GROUPS * tiles[k] / sum)));
    order.resize(n);
    for (int k = 0; k < n; ++k) order[k] = k;
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return m[a] > m[b]; });
    GridShares s{};
    for (int step = 1;; step *= 2) {   // rounded up until there are at most LEVELS different shares
        int l = 0, below = 0;
        s = GridShares{};
        for (int k = n - 1; k >= 0; --k) {   // from the smallest share up
            const int v = (m[order[k]] + step - 1) / step * step;
            if (v == below) continue;
            if (l == GridShares::LEVELS) { l = -1; break; }
            s.grids[l] = k + 1;
            s.width[l++] = v - below;
            below = v;
        }
        if (l >= 0) return s;
    }
}

__host__ __device__ constexpr int nest_frame_cells(int nxe, int nye) {
    return 2 * NEST_FRAME * (nxe + nye - 2 * NEST_FRAME);
}

__device__ __forceinline__ int floor_div(int a, int r) { return a >= 0 ? a / r : -((-a + r - 1) / r); }

// Frame of every patch at time theta in [0, 1) of the coarse step, written to
// the patch buffers pf; the coarse layers n and n+1 are in buffers pc, pc^1.
// Bound by its chain of memory round trips (a few us with 30 k frame cells):
// a row of workgroups per patch (blockIdx.y) makes the descriptor a scalar
// load, and everything a cell may need is loaded before the first use.
template <typename real>
__global__ __launch_bounds__(256) void k_frame(NestArgs<real> n, int pf, int pc, real theta) {
    const NestPatch<real>& d = n.P[blockIdx.y];
    constexpr int G = NEST_FRAME;
    const int nxe = d.nxe, nye = d.nye;
    int m = blockIdx.x * 256 + threadIdx.x, fi, fj;
    if (m >= nest_frame_cells(nxe, nye)) return;
    if (m < G * nxe) {
        fj = m / nxe; fi = m % nxe;
    } else if (m < 2 * G * nxe) {
        m -= G * nxe; fj = nye - G + m / nxe; fi = m % nxe;
    } else {
        m -= 2 * G * nxe;
        fj = G + m / (2 * G);
        const int c = m % (2 * G);
        fi = c < G ? c : nxe - 2 * G + c;
    }
    const int ci = d.ci0 + floor_div(fi - G, n.r), cj = d.cj0 + floor_div(fj - G, n.r);
    const int gc = cj * n.nx + ci, gf = fj * nxe + fi;
    // at theta = 0 the frame is layer n alone (layer n+1 is not computed yet):
    // both terms take layer n's value
    const int pn = theta > real(0) ? pc ^ 1 : pc;
    const real h0 = n.Hc[pc][gc], h1 = n.Hc[pn][gc], x0 = n.Qxc[pc][gc], x1 = n.Qxc[pn][gc];
    const real y0 = n.Qyc[pc][gc], y1 = n.Qyc[pn][gc], bc = n.bc[gc], bf = d.bf[gf];
    const real u = real(1) - theta;
    const real Hm = u * h0 + theta * h1;
    const bool w = Hm > n.eps;
    const real eta = Hm + bc;
    const real Hf = w ? rmax(real(0), eta - bf) : real(0);
    d.Hf[pf][gf] = Hf;
    // the coarse velocity carried by the fine depth (not the coarse
    // discharge, which on a high spot of the fine bed would be a fast film)
    d.Qxf[pf][gf] = w ? Hf * Mth<real>::div(u * x0 + theta * x1, Hm) : real(0);
    d.Qyf[pf][gf] = w ? Hf * Mth<real>::div(u * y0 + theta * y1, Hm) : real(0);
}

// Sums of the r x r fine cells from offset g0 on, row by row.  N loads per
// field are under way together (past the last cell it is loaded again and 0
// added, which leaves a sum unchanged: none is -0).
template <typename real, int N>
__device__ __forceinline__ void block_sums(const NestPatch<real>& d, int pf, int r, int g0, double& sH, double& sX,
                                           double& sY) {
    int jj = 0, ii = 0;
    for (int m0 = 0; m0 < r * r; m0 += N) {
        real h[N], x[N], y[N];
#pragma unroll
        for (int q = 0; q < N; ++q) {
            const int g = g0 + jj * d.nxe + ii;
            h[q] = d.Hf[pf][g]; x[q] = d.Qxf[pf][g]; y[q] = d.Qyf[pf][g];
            if (m0 + q + 1 < r * r && ++ii == r) { ii = 0; ++jj; }
        }
#pragma unroll
        for (int q = 0; q < N; ++q) {
            const bool in = m0 + q < r * r;
            sH += in ? (double)h[q] : 0.0;
            sX += in ? (double)x[q] : 0.0;
            sY += in ? (double)y[q] : 0.0;
        }
    }
}

// Restriction of the fine layer (patch buffers pf) into the covered coarse
// cells (row 1 + k of the grid: patch k) and the flux correction of the ring
// cells (row 0), both in coarse buffer po.  Bound by its chains of memory
// round trips: the loads of a fine block and of a ring face's taps go
// together.
template <typename real>
__global__ __launch_bounds__(256) void k_feedback(NestArgs<real> n, int pf, int po) {
    const int t = blockIdx.x * 256 + threadIdx.x;
    const int r = n.r;
    if (blockIdx.y > 0) {
        const NestPatch<real>& d = n.P[blockIdx.y - 1];
        if (t >= d.cw * d.ch) return;
        const int cy = t / d.cw, cx = t % d.cw;
        const int gc = (d.cj0 + cy) * n.nx + d.ci0 + cx;
        // a block whose tiles hold no water at all (depth sums exactly 0, so
        // every depth and discharge is +0) restricts to zero without being read
        const int fx0 = NEST_FRAME + cx * r, fy0 = NEST_FRAME + cy * r;
        const int tx0 = fx0 / d.tx, tx1 = (fx0 + r - 1) / d.tx, ty0 = fy0 / d.ty, ty1 = (fy0 + r - 1) / d.ty;
        if (d.mass[ty0 * d.ntx + tx0] == 0.0 && d.mass[ty0 * d.ntx + tx1] == 0.0 &&
            d.mass[ty1 * d.ntx + tx0] == 0.0 && d.mass[ty1 * d.ntx + tx1] == 0.0) {
            n.Hc[po][gc] = real(0);
            n.Qxc[po][gc] = real(0);
            n.Qyc[po][gc] = real(0);
            return;
        }
        double sH = 0.0, sX = 0.0, sY = 0.0;
        const int g0 = fy0 * d.nxe + fx0;
        if (r > 2) block_sums<real, 16>(d, pf, r, g0, sH, sX, sY);
        else block_sums<real, 4>(d, pf, r, g0, sH, sX, sY);
        // the restricted cell follows the dry rule of every stored layer: no
        // discharge in a cell with H <= eps (the block mean of a few wet fine
        // cells can leave a dry coarse cell)
        const double inv = 1.0 / (double)(r * r);
        const real Hm = (real)(sH * inv);
        const bool w = Hm > n.eps;
        n.Hc[po][gc] = Hm;
        n.Qxc[po][gc] = w ? (real)(sX * inv) : real(0);
        n.Qyc[po][gc] = w ? (real)(sY * inv) : real(0);
        return;
    }
    const int q = t;
    if (q >= n.nring) return;
    const int gc = n.ring_cell[q];
    const real Hc = n.Hc[po][gc], Qxc = n.Qxc[po][gc], Qyc = n.Qyc[po][gc];
    const double led = n.ring_ledger[q];
    real dH = real(0), dQx = real(0), dQy = real(0);
    for (int e = n.ring_off[q]; e < n.ring_off[q + 1]; ++e) {
        const int k = n.ring_face[3 * e], side = n.ring_face[3 * e + 1], idx = n.ring_face[3 * e + 2];
        const NestPatch<real>& d = n.P[k];
        const int nxf = r * d.cw, nyf = r * d.ch;
        const int pc_ = 2 * (d.cw + d.ch), pf_ = 2 * (nxf + nyf);
        const int oc = side == 0 ? idx : side == 1 ? d.ch + idx : side == 2 ? 2 * d.ch + idx : 2 * d.ch + d.cw + idx;
        const int of = side == 0 ? r * idx : side == 1 ? nyf + r * idx
                     : side == 2 ? 2 * nyf + r * idx : 2 * nyf + nxf + r * idx;
        real corr[3], tc[3], fs[3] = {real(0), real(0), real(0)};
#pragma unroll
        for (int c = 0; c < 3; ++c) tc[c] = n.tap[d.ctap + c * pc_ + oc];
        for (int j0 = 0; j0 < r; j0 += 4) {   // (as block_sums)
            real v[3][4];
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int j = 0; j < 4; ++j) v[c][j] = n.tap[d.ftap + c * pf_ + of + min(j0 + j, r - 1)];
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int j = 0; j < 4; ++j) fs[c] += j0 + j < r ? v[c][j] : real(0);
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) corr[c] = (tc[c] - fs[c] / (real)r) * n.ih;
        // the covered box lies east of a W ring cell (its outflow face) and
        // north of an S ring cell
        const real sg = (side == 0 || side == 2) ? real(1) : real(-1);
        dH += sg * corr[0];
        if (side < 2) { dQx += sg * corr[1]; dQy += sg * corr[2]; }
        else { dQy += sg * corr[1]; dQx += sg * corr[2]; }
    }
    const real Hn = Hc + dH;
    const real Hcl = rmax(Hn, real(0));
    n.ring_ledger[q] = led + (double)(Hcl - Hn) * n.h2;
    const bool w = Hcl > n.eps;
    // momentum weight: 0 up to NEST_MOMENTUM_DEPTH, 1 from twice that,
    // linear between (continuous: rounding cannot flip it)
    const real wm = rmin(real(1), rmax(real(0), Hcl / (real)NEST_MOMENTUM_DEPTH - real(1)));
    n.Hc[po][gc] = Hcl;
    n.Qxc[po][gc] = w ? Qxc + wm * dQx : real(0);
    n.Qyc[po][gc] = w ? Qyc + wm * dQy : real(0);
}

// CFL speed of the new coarse layer (buffers of a's input) at cell (gx, gy);
// 0 for a dry cell.
template <typename real>
__device__ real region_speed(const Args<real>& a, int gx, int gy) {
    const real eps = a.eps;
    real Hs[5], ux[5], uy[5];
    const real cf = a.cf[gy * a.nx + gx];
    const int ox[5] = {0, -1, 1, 0, 0}, oy[5] = {0, 0, 0, -1, 1};
#pragma unroll
    for (int q = 0; q < 5; ++q) {
        int fx = 0, fy = 0;
        const int x = mirror(gx + ox[q], a.nx, fx), y = mirror(gy + oy[q], a.ny, fy);
        const int gi = y * a.nx + x;
        const real H = a.Hi[gi];
        real qx = a.Qxi[gi], qy = a.Qyi[gi];
        if (fx & 1) qx = -qx;
        if (fy & 1) qy = -qy;
        const bool wq = H > eps;
        Hs[q] = H;
        ux[q] = wq ? Mth<real>::div(qx, H) : real(0);
        uy[q] = wq ? Mth<real>::div(qy, H) : real(0);
    }
    if (!(Hs[0] > eps)) return real(0);
    Nb4<real> nb;
#pragma unroll
    for (int q = 0; q < 4; ++q) { nb.ux[q] = ux[q + 1]; nb.uy[q] = uy[q + 1]; nb.w[q] = Hs[q + 1] > eps; }
    real fx, fy;
    soft_forces(a, Hs[0], ux[0], uy[0], nb, fx, fy);
    return cfl_speed(a, Hs[0], cf, ux[0], uy[0], fx, fy);
}

// Lengths of the next coarse step (tc, rounded to the stencil type) and of
// its r substeps; the hydrograph volume of the coarse step follows its clock.
template <typename real>
__device__ void set_nest_steps(const Args<real>& a, const NestArgs<real>& n, double tc) {
    tc = (double)(real)tc;
    set_next_step(a, a.ctrl, tc);
    const double tf = (double)(real)(tc / (double)n.r);
    for (int k = 0; k < n.np; ++k) {
        Ctrl* p = n.P[k].ctrl;
        p->tau = tf;
        p->dV = 0.0;
        p->sdepth = 0.0;
    }
}

// Set the next steps from the host: tc > 0 held, tc = 0 the CFL rule of the
// current layers (speeds recorded by the last coarse step).
template <typename real>
__global__ void k_nest_set_dt(Args<real> a, NestArgs<real> n, double tc) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    if (!(tc > 0.0)) {
        tc = cfl_tau_of(a, a.ctrl->speed);
        for (int k = 0; k < n.np; ++k) tc = fmin(tc, (double)n.r * n.P[k].ctrl->tau_cfl);
    }
    set_nest_steps(a, n, tc);
}

// Time steps of the next coarse step and its substeps; errors of any grid
// stop all of them.  `slot` is the coarse list slot of the next step.  Run
// by the first wave of a workgroup (threads 0..63), with every read of the
// control blocks issued before the first write (two memory round trips, not
// one per field and patch): lane k < np reads patch k's CFL step and error
// (NestReads, which nothing writes while the closing kernels run: they are
// read when those start), lane g < NSEG the coarse list's segment counter g;
// lane 0 then writes the coarse control block and lane k patch k's steps.
// With `region`, s_lane is a speed maximum gathered besides the control
// block's, per lane (0 where there is none).
struct NestReads {
    Ctrl* pc;
    double speed, prep, t, tcf;
    int cerr, perr;
};
template <typename real>
__device__ __forceinline__ NestReads nest_reads(const Args<real>& a, const NestArgs<real>& n) {
    const int lane = threadIdx.x & 63;
    const Ctrl* const c = a.ctrl;
    NestReads v;
    v.pc = lane < n.np ? n.P[lane].ctrl : nullptr;
    v.speed = c->speed;
    v.prep = prep_speed(a.ctrl, real(0));
    v.t = c->t;
    v.cerr = c->err;
    v.tcf = v.pc ? (double)n.r * v.pc->tau_cfl : __builtin_inf();
    v.perr = v.pc ? v.pc->err : 0;
    return v;
}
template <typename real>
__device__ void nest_tau_rule(const Args<real>& a, const NestArgs<real>& n, const NestReads& v, int slot, bool region,
                              double s_lane) {
    const int lane = threadIdx.x & 63;
    Ctrl *const c = a.ctrl, *const pc = v.pc;
    const double speed = v.speed, prep = v.prep, t = v.t, tcf = v.tcf;
    const int cerr = v.cerr, perr = v.perr;
    const int nseg = a.skip && lane < NSEG ? a.hot[hot_seg(slot, lane)] : 0;
    // the rule: tau_c = min(CFL step of the coarse speeds, r * CFL step of
    // every patch), unless held; min and max are exact in any order
    double S = s_lane, tp = tcf;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        S = fmax(S, __shfl_xor(S, o, 64));
        tp = fmin(tp, __shfl_xor(tp, o, 64));
    }
    S = region ? fmax(fmax(speed, prep), S) : fmax(speed, prep);
    const double tc = fmin(cfl_tau_of(a, S), tp);
    const double tcr = (double)(real)(n.hold > 0.0 ? n.hold : tc);
    // the coarse step's scalars (set_next_step's rule) and the substeps'
    const bool bad_step = !(tcr >= a.tau_min) || !(tcr < __builtin_inf());
    double dV = 0.0;
    if (a.nin_h2 > 0.0 && tcr < __builtin_inf())
        dV = hydro_volume(a.q_base, a.q_peak, a.t_peak, a.sigma_t, t, tcr);
    const double tf = (double)(real)(tcr / (double)n.r);
    // the coarse grid's error after the step check, else the first patch's
    int e = bad_step ? -5 : cerr;
    const unsigned long long pm = __ballot(perr != 0);
    const int pe = __shfl(perr, pm ? __ffsll((long long)pm) - 1 : 0, 64);
    if (!e) e = pe;
    int sg[NSEG];
#pragma unroll
    for (int g = 0; g < NSEG; ++g) sg[g] = __shfl(nseg, g, 64);
    // writes
    if (lane == 0) {
        c->prep_speed = 0ull;
        c->speed = S;
        c->tau = tcr;
        c->dV = dV;
        c->sdepth = a.nin_h2 > 0.0 ? (double)(real)(dV / a.nin_h2) : 0.0;
        if (a.skip) close_segments_from(c, sg, slot);
        if (e) { c->err = e; c->err_gate = e; }
    }
    if (pc) {
        pc->tau = tf;
        pc->dV = 0.0;
        pc->sdepth = 0.0;
        if (e) pc->err_gate = e;
    }
}

// The close of a coarse step without feedback: the step rule (first wave
// of block 0) and the taps cleared for the next coarse step (every thread,
// striding; ntap = 0 leaves them).
template <typename real>
__global__ void k_nest_tau(Args<real> a, NestArgs<real> n, int slot, int ntap) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < ntap; i += gridDim.x * blockDim.x) n.tap[i] = real(0);
    if (blockIdx.x != 0 || threadIdx.x >= 64) return;
    nest_tau_rule(a, n, nest_reads(a, n), slot, false, 0.0);
}

// The close of a two-way coarse step, one launch after k_feedback (a row of
// workgroups of 256 threads per patch, at most about NEST_CLOSE_GRID, each
// striding over the work): the CFL speed of the new coarse layer on the cells the feedback can change;
// the tiles round the covered boxes put on the coarse list of the next step
// (list `slot`, generation of that list), so that the cells the feedback
// changed are stepped and both buffers of the pair stay consistent; the taps
// cleared for the next coarse step.  The last workgroup to finish sets the
// next steps (k_nest_tau's rule).  Completion uses the coarse grid's group
// words, which are zero between two of its step launches: each workgroup's
// speed maximum and arrival go to its group's words by atomics, the arrival
// issued only once the maximum has returned (so are the workgroup's
// appends, whose results feed its list writes before the barrier), and the
// last arrival of the last group reads and clears them.
// Bound by its chain of round trips, not by bytes: one cell per thread with
// all its loads together, the appends by the workgroups from the last on
// (the region's cells lie with the first of each row), and what the step
// rule reads of the control blocks loaded at the start.
constexpr int NEST_CLOSE_GRID = 1024;
template <typename real>
__global__ __launch_bounds__(256) void k_nest_close(Args<real> a, NestArgs<real> n, const int* rects,
                                                    const int* force, int nforce, int ntap, int slot) {
    constexpr int NT = 256;
    __shared__ real red[NT / 64];
    __shared__ int s_last;
    const int tid = threadIdx.x, G = gridDim.x * gridDim.y, b = blockIdx.y * gridDim.x + blockIdx.x, grp = b % NSEG;
    const int* const R = rects + 4 * blockIdx.y;   // x0, y0, x1, y1: the covered box widened by 2 cells
    const int rx0 = R[0], ry0 = R[1], rw = R[2] - rx0, cells = rw * (R[3] - ry0);
    NestReads reads = {};
    if (tid < 64) reads = nest_reads(a, n);
    real vmax = real(0);
    for (int t = blockIdx.x * NT + tid; t < cells; t += gridDim.x * NT)
        vmax = rmax(vmax, region_speed(a, rx0 + t % rw, ry0 + t / rw));
    const int gen = (int)a.ctrl->step + 1;
    // whole workgroups take each round (the append votes per wave)
    for (int t0 = (G - 1 - b) * NT; t0 < nforce; t0 += G * NT)
        append_tiles(t0 + tid < nforce ? force[t0 + tid] : -1, 0, 0, gen, a.stamp, a.lists, a.hot, a.ntiles, slot,
                     grp);
    for (int t = b * NT + tid; t < ntap; t += G * NT) n.tap[t] = real(0);
    vmax = wave_max(vmax);
    if ((tid & 63) == 0) red[tid >> 6] = vmax;
    __syncthreads();
    unsigned long long* const h64 = reinterpret_cast<unsigned long long*>(a.hot);
    if (tid == 0) {
        real vm = real(0);
        for (int q = 0; q < NT / 64; ++q) vm = rmax(vm, red[q]);
        const unsigned long long sp = atomicMax(&h64[hot_spd(grp) / 2], (unsigned long long)__double_as_longlong((double)vm));
        const int in_grp = (G - grp + NSEG - 1) / NSEG, ngrp = G < NSEG ? G : NSEG;
        bool last = false;
        if (sp != ~0ull) {        // always (no speed has these bits): waits for the maximum
            const unsigned long long old = atomicAdd(&h64[hot_cnt(grp) / 2], 1ull);
            if ((int)old == in_grp - 1)
                last = atomicAdd((unsigned*)&a.hot[hot_done(NSEG)], 1u) == (unsigned)(ngrp - 1);
        }
        s_last = last;
    }
    __syncthreads();
    if (!s_last) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    if (tid < 64) {
        const double sg = tid < NSEG ? __longlong_as_double((long long)h64[hot_spd(tid) / 2]) : 0.0;
        nest_tau_rule(a, n, reads, slot, true, sg);
        if (tid < NSEG) { h64[hot_cnt(tid) / 2] = 0ull; h64[hot_spd(tid) / 2] = 0ull; }
        if (tid == 0) a.hot[hot_done(NSEG)] = 0;
    }
}

// Fixed-order sum of a field (volume of the nested solution): per-block
// partials, then k_sum_tiles.
template <typename real>
__global__ void k_field_partials(const real* f, int n, int chunk, double* part) {
    __shared__ double red[256 / 64];
    const int b = blockIdx.x, i0 = b * chunk, i1 = min(n, i0 + chunk);
    double s = 0.0;
    for (int i = i0 + (int)threadIdx.x; i < i1; i += blockDim.x) s += (double)f[i];
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double v = 0.0;
        for (int q = 0; q < (int)blockDim.x / 64; ++q) v += red[q];
        part[b] = v;
    }
}

}  // namespace swe
