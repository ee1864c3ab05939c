// HIP kernels of the CCZ4 FD4 hot path for gfx950 (MI355X).
//
// State layout: per leaf patch, slot-major boxes of 15 x 15 x 16 doubles (see ccz4.h).
// Every kernel maps one thread to one cell (or one halo cell) so that consecutive lanes walk
// the contiguous x rows of a box.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ccz4_algebra.hpp"
#include "ccz4_device.hpp"
#include "ccz4_kernels.hpp"
#include "ccz4_rhs_lds.hpp"
#include "ccz4_rhs_phased.hpp"

namespace ccz4 {

// ------------------------------------------------------------------ initial data
// Closed forms of the three scenarios at a point; the first-order auxiliaries are the
// analytic derivatives (A = d alpha, B = d beta, D = d gt / 2, P = d phi).
__device__ void init_point(int scen, const double *sp, double x, double y, double z, double *q)
{
    for (int v = 0; v < NV; ++v) q[v] = 0.0;
    if (scen == 0) {
        const double A = sp[0], kk = sp[1];
        const double w = kk * M_PI;
        const double Hh = 1.0 - A * sin(w * x);
        const double dH = -A * w * cos(w * x);
        const double sq = sqrt(Hh);
        const double Kxx = dH / (2.0 * sq);
        const double Hm13 = pow(Hh, -1.0 / 3.0);
        q[SG + 0] = Hh * Hm13;
        q[SG + 3] = Hm13;
        q[SG + 5] = Hm13;
        q[SALPHA] = sq;
        q[SPHI] = pow(Hh, -1.0 / 6.0);
        q[SAT + 0] = (2.0 / 3.0) * Hm13 * Kxx;
        q[SAT + 3] = -(1.0 / 3.0) * Hm13 / Hh * Kxx;
        q[SAT + 5] = q[SAT + 3];
        q[SK] = Kxx / Hh;
        q[SGHAT + 0] = (2.0 / 3.0) * Hm13 * Hm13 / Hh * dH;
        q[SA + 0] = Kxx;
        q[SD + 0] = (1.0 / 3.0) * Hm13 * dH;
        q[SD + 3] = -(1.0 / 6.0) * Hm13 / Hh * dH;
        q[SD + 5] = q[SD + 3];
        q[SP + 0] = -(1.0 / 6.0) * q[SPHI] / Hh * dH;
        return;
    }
    q[SG + 0] = q[SG + 3] = q[SG + 5] = 1.0;
    if (scen == 1) {
        const double M = sp[0];
        const double rx = x - sp[1], ry = y - sp[2], rz = z - sp[3];
        const double r = sqrt(rx * rx + ry * ry + rz * rz);
        const double psi = 1.0 + 0.5 * M / r;
        const double ipsi = 1.0 / psi;
        const double f = 0.5 * M / (r * r * r);  // -d_k psi = f x_k
        const double phi = ipsi * ipsi;
        q[SPHI] = phi;
        const double pk = 2.0 * phi * ipsi * f;  // d_k phi = -2 psi^-3 d_k psi
        q[SP + 0] = pk * rx;
        q[SP + 1] = pk * ry;
        q[SP + 2] = pk * rz;
        const int lapse = (int)sp[4];
        if (lapse == 0) {
            q[SALPHA] = phi;
            q[SA + 0] = q[SP + 0];
            q[SA + 1] = q[SP + 1];
            q[SA + 2] = q[SP + 2];
        } else {
            const double as = (2.0 - psi) * ipsi;   // (1 - M/2r)/(1 + M/2r)
            const double wgt = lapse == 1 ? 0.5 : 1.0;
            q[SALPHA] = lapse == 1 ? 0.5 * (as + 1.0) : as;
            const double ak = wgt * 2.0 * phi * f;  // d_k alpha_s = -2 psi^-2 d_k psi
            q[SA + 0] = ak * rx;
            q[SA + 1] = ak * ry;
            q[SA + 2] = ak * rz;
        }
        return;
    }
    // two Brill-Lindquist holes with Bowen-York curvature
    double psi = 1.0, dpsi[3] = {0.0, 0.0, 0.0}, Ah[6] = {0, 0, 0, 0, 0, 0};
    for (int h = 0; h < 2; ++h) {
        const double *s = sp + 7 * h;
        const double d[3] = {x - s[1], y - s[2], z - s[3]};
        const double r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
        const double r = sqrt(r2);
        const double n[3] = {d[0] / r, d[1] / r, d[2] / r};
        psi += 0.5 * s[0] / r;
        for (int i = 0; i < 3; ++i) dpsi[i] -= 0.5 * s[0] * d[i] / (r2 * r);
        const double Pn = s[4] * n[0] + s[5] * n[1] + s[6] * n[2];
        const double c = 1.5 / r2;
        for (int i = 0; i < 3; ++i)
            for (int j = i; j < 3; ++j)
                Ah[sym(i, j)] += c * (s[4 + i] * n[j] + s[4 + j] * n[i] - ((i == j) - n[i] * n[j]) * Pn);
    }
    const double ipsi = 1.0 / psi;
    const double phi = ipsi * ipsi;
    const double ip6 = phi * phi * phi;
    q[SPHI] = phi;
    q[SALPHA] = phi;
    for (int i = 0; i < 3; ++i) {
        q[SP + i] = -2.0 * phi * ipsi * dpsi[i];
        q[SA + i] = q[SP + i];
    }
    for (int s = 0; s < 6; ++s) q[SAT + s] = ip6 * Ah[s];
}

// interior cells, projected
__global__ __launch_bounds__(256) void k_init(double *__restrict__ Q, const PatchGeom *__restrict__ geom, int32_t npatch,
                                              int32_t scen, InitArgs a)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)npatch * NCELL) return;
    const int p = (int)(t / NCELL), c = (int)(t % NCELL);
    const int x = c % 9 + 3, y = (c / 9) % 9 + 3, z = c / 81 + 3;
    const PatchGeom g = geom[p];
    double q[NV];
    init_point(scen, a.sp, g.org[0] + (x - 2.5) * g.dx[0], g.org[1] + (y - 2.5) * g.dx[1],
               g.org[2] + (z - 2.5) * g.dx[2], q);
    project_cell(q);
    double *Qp = Q + (int64_t)p * PS + boff(x, y, z);
    for (int v = 0; v < NV; ++v) Qp[(int64_t)v * CS] = q[v];
}

// Sommerfeld ghosts (evolved, not projected) and the background they hold, one work-group per face.
// With regrid tasks, a leaf that was copied keeps the ghosts it brought and only its background is set.
__global__ __launch_bounds__(256) void k_init_ghosts(double *__restrict__ Q, const PatchGeom *__restrict__ geom,
                                                     const BoundaryFace *__restrict__ bf, double *__restrict__ bg,
                                                     int32_t nbf, const RegridTask *__restrict__ tasks, int32_t scen,
                                                     InitArgs a)
{
    const int fi = blockIdx.x, idx = threadIdx.x;
    if (fi >= nbf || idx >= NFACE) return;
    const BoundaryFace f = bf[fi];
    int L, t1, t2;
    slab_coords(f.axis, idx, L, t1, t2);
    const int o = slab_off(f.axis, ghost_c(f.side, L), t1, t2);
    const int x = o % XS, y = (o / YS) % NBX, z = o / ZS;
    const PatchGeom g = geom[f.patch];
    double q[NV];
    init_point(scen, a.sp, g.org[0] + (x - 2.5) * g.dx[0], g.org[1] + (y - 2.5) * g.dx[1],
               g.org[2] + (z - 2.5) * g.dx[2], q);
    double *B = bg + (int64_t)f.bg * NV * NFACE + idx;
    for (int v = 0; v < NV; ++v) B[v * NFACE] = q[v];
    if (tasks && tasks[f.patch].kind == RG_COPY) return;
    double *Qp = Q + (int64_t)f.patch * PS + o;
    for (int v = 0; v < NV; ++v) Qp[(int64_t)v * CS] = q[v];
}

// ------------------------------------------------------------------ halo fill
// P_parallel row F (0..26) -> (first coarse index, weights w0, w1)
__device__ __forceinline__ void ppar(int F, int &l, double &w0, double &w1)
{
    // u = (F + 1/2)/3 - 1/2 = (2F - 2)/6 ; l = clamp(floor(u), 0, 7)
    const int num = F - 1;  // u = num / 3
    int lf = num >= 0 ? num / 3 : -1;
    l = lf < 0 ? 0 : (lf > 7 ? 7 : lf);
    const double u = (double)num / 3.0;
    w1 = u - l;
    w0 = 1.0 - w1;
}

// Same-level faces: a work-group takes two slots of one leaf.  Its lanes read the leaf's interior once
// and copy it into the neighbours' y and z face halos; the x halos, three cells at either end of the
// leaf's own rows, are gathered, both ends of a row by one instruction.  Sources are interior cells and
// destinations ghosts, each written by one lane.  Bound by the partial lines that are written (24 and
// 72 of 128 bytes: 189 a slot and leaf, which memory reads and writes back): on 16^3 leaves 3.93 ms by
// one block per face and eight slots -> 2.44 ms; every face gathered 2.79 ms, every face copied out
// 2.47 ms, y and z copies not streamed past the caches 2.64 ms, eight slots a work-group 2.50 ms.
constexpr int COPY_LANES = 768, COPY_SLOTS = 2, COPY_BATCHES = (NV + COPY_SLOTS - 1) / COPY_SLOTS;

__global__ __launch_bounds__(COPY_LANES) void k_copy_faces(double *__restrict__ Q, const int32_t *__restrict__ nbr,
                                                           int32_t npatch)
{
    const int64_t lb = xcd_logical_block(blockIdx.x, gridDim.x);
    const int p = (int)(lb / COPY_BATCHES);
    if (p >= npatch) return;
    const int v0 = (int)(lb % COPY_BATCHES) * COPY_SLOTS;
    double *Qp = Q + (int64_t)p * PS + (int64_t)v0 * CS;
    const int i = (int)threadIdx.x;
    int64_t pd[3] = {0, 0, 0};
    const int x = i % 9 + 3, y = (i / 9) % 9 + 3, z = i / 81 + 3, o = boff(x, y, z);
    if (i < NCELL) push_offsets(nbr, p, x, y, z, o, pd, 6);
    const bool push = pd[1] != 0 || pd[2] != 0;
    // x ghost cell k (0..2 low, 3..5 high) of row i / 6
    const int row = i / 6, k = i % 6, og = boff(k < 3 ? k : k + 9, row % 9 + 3, row / 9 + 3);
    const int q = i < 6 * PN * PN ? nbr[6 * p + (k < 3 ? 0 : 1)] : -1;
    const int64_t xd = (int64_t)(q - p) * PS + og + (k < 3 ? 9 : -9);
    double own[COPY_SLOTS], gh[COPY_SLOTS];
#pragma unroll
    for (int j = 0; j < COPY_SLOTS; ++j)
        if (v0 + j < NV) {
            if (push) own[j] = Qp[j * CS + o];
            if (q >= 0) gh[j] = Qp[j * CS + xd];
        }
#pragma unroll
    for (int j = 0; j < COPY_SLOTS; ++j)
        if (v0 + j < NV) {
            if (q >= 0) Qp[j * CS + og] = gh[j];
#pragma unroll
            for (int a = 1; a < 3; ++a)
                if (pd[a] != 0) __builtin_nontemporal_store(own[j], Qp + j * CS + o + pd[a]);
        }
}

// The other kinds: one block per (face task, batch of eight slots), one thread per slab cell.  Bound by the
// partial lines that a level pair's fills touch, and by the loads in flight.  The higher-order prolongation
// keeps 27 offsets and weights for all its slots, 198 registers: two waves per SIMD.  At four it spills 72
// of them, and then one slot a block, which forms them for every slot anew, takes longest (144 coarse
// faces, 0.40 ms at two waves; at four 1.08 ms, and 1.90 ms with one slot a block).  The operators of two
// and nine points need few registers; more than four waves per SIMD only press on the caches (144 and 480
// coarse faces, 0.350 and 1.11 ms; six waves 0.358 and 1.24 ms, four slots a block 0.376 and 1.21 ms).
constexpr int FILL_SLOTS = 8;

template <int HIGHER>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(HIGHER ? 2 : 4, HIGHER ? 2 : 4))) void k_fill(
    double *__restrict__ Q, const FaceTask *__restrict__ tasks, int32_t ntask, int32_t v_first, int32_t v_end)
{
    constexpr int SLOTS = FILL_SLOTS;
    const int ti = blockIdx.x;
    const int idx = threadIdx.x;
    if (ti >= ntask || idx >= NFACE) return;
    // blockIdx.y picks the batch, so that a task's slots are filled in parallel
    const int v_lo = v_first + (int)blockIdx.y * SLOTS, v_hi = min(v_lo + SLOTS, v_end);
    const FaceTask tk = tasks[ti];
    int L, t1, t2;
    slab_coords(tk.axis, idx, L, t1, t2);
    double *dst = Q + (int64_t)tk.patch * PS + slab_off(tk.axis, ghost_c(tk.side, L), t1, t2);
    if (tk.kind == (HIGHER ? FK_RESTRICT : FK_NEUMANN)) {
        // copies; with the higher-order operators the restriction is one too: coarse ghost c_{2+L}
        // takes the fine cell with the same centre, tangentially the middle of the three fine
        // cells under it, along the normal the fine interior depth 3L - 1
        const int F1 = 3 * t1 + 1, F2 = 3 * t2 + 1;
        const double *src = HIGHER
                                ? Q + (int64_t)tk.src[(F2 / 9) * 3 + F1 / 9] * PS +
                                      slab_off(tk.axis, depth_c(-tk.side, 3 * L - 1), F1 % 9, F2 % 9)
                                : Q + (int64_t)tk.patch * PS + slab_off(tk.axis, depth_c(tk.side, 1), t1, t2);
        double r[SLOTS];
#pragma unroll
        for (int i = 0; i < SLOTS; ++i) r[i] = (v_lo + i < v_hi) ? src[(v_lo + i) * CS] : 0.0;
#pragma unroll
        for (int i = 0; i < SLOTS; ++i)
            if (v_lo + i < v_hi) dst[(v_lo + i) * CS] = r[i];
    } else if (tk.kind == FK_RESTRICT) {
        // coarse ghost c_{2+L}; fine interior layers f3..f5 = depth 1..3 from the kid's face -side;
        // R_perp rows (1/3,1/3,1/3), (0,-2,3), (0,-5,6) over (f3,f4,f5); R_avg over 3x3 fine cells
        double wf[3];
        if (L == 1) { wf[0] = wf[1] = wf[2] = 1.0 / 3.0; }
        else if (L == 2) { wf[0] = 0.0; wf[1] = -2.0; wf[2] = 3.0; }
        else { wf[0] = 0.0; wf[1] = -5.0; wf[2] = 6.0; }
        const int k1 = (3 * t1) / 9, k2 = (3 * t2) / 9;
        const double *kid = Q + (int64_t)tk.src[k2 * 3 + k1] * PS;
        const int f1 = (3 * t1) % 9, f2 = (3 * t2) % 9;
        int off[3][9];
        for (int m = 0; m < 3; ++m)
            for (int b2 = 0; b2 < 3; ++b2)
                for (int b1 = 0; b1 < 3; ++b1)
                    off[m][b2 * 3 + b1] = slab_off(tk.axis, depth_c(-tk.side, m + 1), f1 + b1, f2 + b2);
        for (int v = v_lo; v < v_hi; ++v) {
            double acc = 0.0;
            for (int m = 0; m < 3; ++m) {
                if (wf[m] == 0.0) continue;
                double sum = 0.0;
#pragma unroll
                for (int n = 0; n < 9; ++n) sum += kid[v * CS + off[m][n]];
                acc += wf[m] * (sum * (1.0 / 9.0));
            }
            dst[v * CS] = acc;
        }
    } else if constexpr (HIGHER) {  // FK_PROLONG
        // three-point Lagrange quadratics along every axis.  Tangentially fine cell F sits at
        // coarse coordinate u = (F + 1/2)/3 - 1/2, taken from the coarse centres l-1, l, l+1 with
        // l the nearest one kept in 1..7; along the normal fine ghost L sits s = 1/2 - (L - 1/2)/3
        // coarse cells from c2 towards the face, taken from c1, c2 and the restricted c3.
        const double *cp = Q + (int64_t)tk.src[0] * PS;
        const double sn = 0.5 - (L - 0.5) / 3.0;
        const double wn[3] = {sn * (sn - 1.0) / 2.0, 1.0 - sn * sn, sn * (sn + 1.0) / 2.0};
        const int cn[3] = {depth_c(-tk.side, 2), depth_c(-tk.side, 1), ghost_c(-tk.side, 1)};
        int j[2];
        double w[2][3];
        const int F[2] = {9 * tk.o1 + t1, 9 * tk.o2 + t2};
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            const double u = (F[d] + 0.5) / 3.0 - 0.5;
            int l = (int)floor(u + 0.5);
            l = l < 1 ? 1 : (l > 7 ? 7 : l);
            const double s = u - l;
            j[d] = l;
            w[d][0] = s * (s - 1.0) / 2.0;
            w[d][1] = 1.0 - s * s;
            w[d][2] = s * (s + 1.0) / 2.0;
        }
        for (int v = v_lo; v < v_hi; ++v) {
            const double *c = cp + v * CS;
            double acc = 0.0;
#pragma unroll
            for (int kn = 0; kn < 3; ++kn)
#pragma unroll
                for (int k2 = 0; k2 < 3; ++k2)
#pragma unroll
                    for (int k1 = 0; k1 < 3; ++k1)
                        acc += wn[kn] * w[1][k2] * w[0][k1] * c[slab_off(tk.axis, cn[kn], j[0] - 1 + k1, j[1] - 1 + k2)];
            dst[v * CS] = acc;
        }
    } else {  // FK_PROLONG
        // fine ghost L -> f_{3-L}; P_perp rows over coarse (c0..c5): f0 = c1/3 + 2c2/3, f1 = c2,
        // f2 = 2c2/3 + c3/3; c0..c2 coarse interior depth 3..1 from the coarse face -side, c3..c5
        // its ghosts 1..3
        const double *cp = Q + (int64_t)tk.src[0] * PS;
        int cA[2];
        double wA[2];
        if (L == 3) { cA[0] = depth_c(-tk.side, 2); wA[0] = 1.0 / 3.0; cA[1] = depth_c(-tk.side, 1); wA[1] = 2.0 / 3.0; }
        else if (L == 2) { cA[0] = depth_c(-tk.side, 1); wA[0] = 1.0; cA[1] = cA[0]; wA[1] = 0.0; }
        else { cA[0] = depth_c(-tk.side, 1); wA[0] = 2.0 / 3.0; cA[1] = ghost_c(-tk.side, 1); wA[1] = 1.0 / 3.0; }
        int l1, l2;
        double a0, a1, b0, b1;
        ppar(9 * tk.o1 + t1, l1, a0, a1);
        ppar(9 * tk.o2 + t2, l2, b0, b1);
        int off[2][4];
        for (int m = 0; m < 2; ++m) {
            off[m][0] = slab_off(tk.axis, cA[m], l1, l2);
            off[m][1] = slab_off(tk.axis, cA[m], l1 + 1, l2);
            off[m][2] = slab_off(tk.axis, cA[m], l1, l2 + 1);
            off[m][3] = slab_off(tk.axis, cA[m], l1 + 1, l2 + 1);
        }
        for (int v = v_lo; v < v_hi; ++v) {
            const double *c = cp + v * CS;
            double acc = 0.0;
            for (int m = 0; m < 2; ++m) {
                if (wA[m] == 0.0) continue;
                const double r0 = a0 * c[off[m][0]] + a1 * c[off[m][1]];
                const double r1 = a0 * c[off[m][2]] + a1 * c[off[m][3]];
                acc += wA[m] * (b0 * r0 + b1 * r1);
            }
            dst[v * CS] = acc;
        }
    }
}

// ------------------------------------------------------------------ right-hand side
#ifndef CCZ4_RHS_WPE
#define CCZ4_RHS_WPE 1
#endif

template <typename T, int LOP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(CCZ4_RHS_WPE))) void k_rhs(const double *__restrict__ Q, double *__restrict__ K,
                                             const PatchGeom *__restrict__ geom, int32_t npatch,
                                             RhsParams prm, int32_t linear, const int32_t *__restrict__ order)
{
    const int64_t lb = linear ? (int64_t)blockIdx.x : xcd_logical_block(blockIdx.x, gridDim.x);
    if (lb / 3 >= npatch || threadIdx.x >= 243) return;
    const int p = order[lb / 3];
    const int c = (int)(lb % 3) * 243 + threadIdx.x;
    const PatchGeom g = geom[p];
    CellRef cr;
    cr.qb = Q + (int64_t)p * PS;
    cr.kb = K + (int64_t)p * PS;
    cr.o = boff(c % 9 + 3, (c / 9) % 9 + 3, c / 81 + 3);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        cr.i12[a] = 1.0 / (12.0 * g.dx[a]);
        cr.koc[a] = prm.ko_eps / (64.0 * g.dx[a]);
    }
    cr.adv = prm.advection;
    RhsSink<LOP> snk;
    snk.so = prm.formulation;
    rhs_cell_phased<T>(cr, prm, snk);
}

// Fused stage: the right-hand side of Qs folded slot by slot into stage s of RK4 (two-register
// form) on the interior cells, with the projection of Q^{n+1} at s = 3.  Qs is read through the
// stencils, Qn and acc pointwise; Qnext must differ from Qs (other cells still read Qs).
template <int L>
struct StageSink {
    static constexpr int LOP = L;  // lopsided advection stencils in the phase functions
    const double *__restrict__ qn;
    double *__restrict__ acc;
    double *__restrict__ qx;
    int s;
    int so;  // second-order formulation: the auxiliaries are left alone (reconstructed afterwards)
    double dt;
    double carry[12];  // s = 3: gt_ij and At_ij of Q^{n+1}, projected in finish()
    int oc;            // the cell's index in a slot of the accumulator (acc_cell)
    int64_t pd[3];     // offsets (doubles, from this cell) of its copies in same-level neighbours'
                       // face halos of Q_next along each axis, 0 for none

    // Q_next at element e, and its copies in the neighbours' halos (after every stage: this kernel reads
    // them there).  Those into the y and z face halos are streamed past the caches: their rows are
    // partial lines that nothing else writes, and on all but small meshes L2 has evicted them before
    // the next stage comes to them (a step of 125 / 720 / 4096 leaves 1.52 / 7.19 / 40.1 ms, cached 1.53 /
    // 7.30 / 40.9 ms; of 27 leaves 0.65 ms, cached 0.55 ms).  The x-face copies stay cached: they
    // complete lines of the neighbour's own rows in L2.
    __device__ __forceinline__ void out(int64_t e, double val)
    {
        qx[e] = val;
        if (pd[0] != 0) qx[e + pd[0]] = val;
#pragma unroll
        for (int a = 1; a < 3; ++a)
            if (pd[a] != 0) __builtin_nontemporal_store(val, qx + e + pd[a]);
    }

    __device__ __forceinline__ void combine_at(int o, int v, double r)
    {
        if (so && aux_slot(v)) return;
        const int e = v * CS + o;
        if (s == 0) {
            const double q0 = qn[e];
            acc[v * CS + oc] = q0 + (1.0 / 6.0) * dt * r;
            out(e, q0 + 0.5 * dt * r);
        } else if (s < 3) {
            acc[v * CS + oc] = acc[v * CS + oc] + (1.0 / 3.0) * dt * r;
            out(e, qn[e] + (s == 1 ? 0.5 : 1.0) * dt * r);
        } else {
            const double val = acc[v * CS + oc] + (1.0 / 6.0) * dt * r;
            if (v < 6) carry[v] = val;
            else if (v >= SAT && v < SAT + 6) carry[v - SAT + 6] = val;
            else out(e, val);
        }
    }
    __device__ __forceinline__ void put(const CellRef &c, int v, double alg) { combine_at(c.o, v, alg + ko(c, v)); }
    __device__ __forceinline__ void zero(const CellRef &c, int v) { combine_at(c.o, v, 0.0); }
    __device__ __forceinline__ void finish(const CellRef &c) { finish_at(c.o); }
    __device__ __forceinline__ void finish_at(int o)
    {
        if (s != 3) return;
        double q[SAT + 6];
#pragma unroll
        for (int v = 0; v < 6; ++v) {
            q[v] = carry[v];
            q[SAT + v] = carry[6 + v];
        }
        project_cell(q);
#pragma unroll
        for (int v = 0; v < 6; ++v) {
            out(v * CS + o, q[v]);
            out((SAT + v) * CS + o, q[SAT + v]);
        }
    }
};

template <typename T, int LOP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(CCZ4_RHS_WPE))) void k_stage(
    const double *__restrict__ Qs, const double *__restrict__ Qn, double *__restrict__ acc, double *__restrict__ Qx,
    const PatchGeom *__restrict__ geom, int32_t npatch, int32_t nb_slab, RhsParams prm, int32_t s, double dt,
    const BoundaryFace *__restrict__ bf, const double *__restrict__ bg, const int32_t *__restrict__ nbr,
    int32_t paxes, int32_t linear, const int32_t *__restrict__ order)
{
    if ((int32_t)blockIdx.x >= nb_slab) {
        stage_ghost_face((int)blockIdx.x - nb_slab, threadIdx.x, s, dt, Qs, Qn, acc, Qx, geom, bf, bg, prm.shift == 0);
        return;
    }
    const int64_t lb = linear ? (int64_t)blockIdx.x : xcd_logical_block(blockIdx.x, nb_slab);
    if (lb / 3 >= npatch || threadIdx.x >= 243) return;
    const int p = order[lb / 3];
    const int c = (int)(lb % 3) * 243 + threadIdx.x;
    const PatchGeom g = geom[p];
    CellRef cr;
    cr.qb = Qs + (int64_t)p * PS;
    cr.kb = nullptr;
    cr.o = boff(c % 9 + 3, (c / 9) % 9 + 3, c / 81 + 3);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        cr.i12[a] = 1.0 / (12.0 * g.dx[a]);
        cr.koc[a] = prm.ko_eps / (64.0 * g.dx[a]);
    }
    cr.adv = prm.advection;
    StageSink<LOP> snk;
    snk.qn = Qn + (int64_t)p * PS;
    snk.acc = acc + (int64_t)p * PS;
    snk.qx = Qx + (int64_t)p * PS;
    snk.s = s;
    snk.so = prm.formulation;
    snk.dt = dt;
    snk.oc = acc_cell((int)(lb % 3), slab_lane((int)threadIdx.x / 81, ((int)threadIdx.x / 9) % 9, (int)threadIdx.x % 9));
    push_offsets(nbr, p, c % 9 + 3, (c / 9) % 9 + 3, c / 81 + 3, cr.o, snk.pd, paxes);
    rhs_cell_phased<T>(cr, prm, snk);
}

// Sommerfeld ghosts: one thread per (boundary face, slot, ghost cell)
__global__ __launch_bounds__(256) void k_rhs_sommerfeld(const double *__restrict__ Q, double *__restrict__ K,
                                                        const PatchGeom *__restrict__ geom,
                                                        const BoundaryFace *__restrict__ bf,
                                                        const double *__restrict__ bg, int32_t nbf, int32_t frozen)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)nbf * NV * NFACE) return;
    const int fi = (int)(t / (NV * NFACE));
    const int r = (int)(t % (NV * NFACE));
    const int v = r / NFACE;
    const int idx = r % NFACE;
    const BoundaryFace f = bf[fi];
    int L, t1, t2;
    slab_coords(f.axis, idx, L, t1, t2);
    const int cg = ghost_c(f.side, L);
    const int og = slab_off(f.axis, cg, t1, t2);
    double *Kp = K + (int64_t)f.patch * PS + v * CS + og;
    if (v == SK0 || (frozen && frozen_slot(v))) {
        *Kp = 0.0;
        return;
    }
    const int ci = L == 1 ? depth_c(f.side, 1) : ghost_c(f.side, L - 1);
    const int oi = slab_off(f.axis, ci, t1, t2);
    const PatchGeom g = geom[f.patch];
    int cx, cy, cz;
    if (f.axis == 0) { cx = cg; cy = t1 + 3; cz = t2 + 3; }
    else if (f.axis == 1) { cx = t1 + 3; cy = cg; cz = t2 + 3; }
    else { cx = t1 + 3; cy = t2 + 3; cz = cg; }
    const double X = g.org[0] + (cx - 2.5) * g.dx[0];
    const double Y = g.org[1] + (cy - 2.5) * g.dx[1];
    const double Z = g.org[2] + (cz - 2.5) * g.dx[2];
    const double rr = sqrt(X * X + Y * Y + Z * Z);
    const double xn = f.axis == 0 ? X : (f.axis == 1 ? Y : Z);
    const double *Qp = Q + (int64_t)f.patch * PS + v * CS;
    const double qL = Qp[og];
    *Kp = -(rr / (fabs(xn) * g.dx[f.axis])) * (qL - Qp[oi]) - (1.0 / rr) * (qL - bg[(int64_t)f.bg * NV * NFACE + v * NFACE + idx]);
}

__global__ void k_capture_bg(const double *__restrict__ Q, const BoundaryFace *__restrict__ bf,
                             double *__restrict__ bg, int32_t nbf)
{
    const int fi = blockIdx.x;
    if (fi >= nbf) return;
    const int idx = threadIdx.x;
    if (idx >= NFACE) return;
    const BoundaryFace f = bf[fi];
    int L, t1, t2;
    slab_coords(f.axis, idx, L, t1, t2);
    const int og = slab_off(f.axis, ghost_c(f.side, L), t1, t2);
    const double *Qp = Q + (int64_t)f.patch * PS;
    for (int v = 0; v < NV; ++v) bg[(int64_t)f.bg * NV * NFACE + v * NFACE + idx] = Qp[v * CS + og];
}

// ------------------------------------------------------------------ RK4 stage
// Classical RK4 in two-register form at N elements of a lane, e(0..N - 1), negative where there is none.
// Every load comes first: the compiler cannot move a load past the store of another element by itself.
template <int N, typename Element>
__device__ __forceinline__ void rk_combine(int s, double dt, const double *__restrict__ qn, const double *__restrict__ kk,
                                           double *__restrict__ acc, double *__restrict__ qx, Element e)
{
    double k[N], q[N], a[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
        if (e(j) < 0) continue;
        k[j] = kk[e(j)];
        if (s < 3) q[j] = qn[e(j)];
        if (s > 0) a[j] = acc[e(j)];
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
        if (e(j) < 0) continue;
        if (s == 0) {
            acc[e(j)] = q[j] + (1.0 / 6.0) * dt * k[j];
            qx[e(j)] = q[j] + 0.5 * dt * k[j];
        } else if (s < 3) {
            acc[e(j)] = a[j] + (1.0 / 3.0) * dt * k[j];
            qx[e(j)] = s == 1 ? q[j] + 0.5 * dt * k[j] : q[j] + dt * k[j];
        } else {
            qx[e(j)] = a[j] + (1.0 / 6.0) * dt * k[j];
        }
    }
}

// RK4_PARTS work-groups per leaf combine its interior, one cell a lane, a run of slots each, the first with
// the slots that s = 3 projects together; RK4_CHUNKS more for each of its six faces combine the ghosts, where
// the face is a Sommerfeld one (not projected).  Bound by memory, most of it the partial lines written, and on
// few leaves by the chain of a work-group's loads, which is therefore kept to one or two batches.  Stages 0..3
// together on 1 / 27 / 125 / 720 / 4096 leaves: 45 / 96 / 453 / 2560 / 13080 us; 142 / 132 / 493 / 2754 / 13800
// us where the first work-groups took the ghosts too, face by face and slot by slot; 112 / 190 / 519 / 2980 /
// 15120 us by a kernel over all cells and one over all ghosts.
constexpr int RK4_PARTS = 4, RK4_CHUNKS = 4, RK4_LANES = 768;
constexpr int RK4_HEAD = SAT + 6, RK4_REST = (NV - RK4_HEAD) / (RK4_PARTS - 1);
constexpr int RK4_CHUNK = (NV + RK4_CHUNKS - 1) / RK4_CHUNKS;  // slots of a ghost work-group, every third a lane's
static_assert(RK4_HEAD + (RK4_PARTS - 1) * RK4_REST == NV && RK4_LANES >= 3 * NFACE, "slots of the parts");

template <int GHOSTS>
__global__ __launch_bounds__(RK4_LANES) void k_rk4(int32_t s, double dt, const double *__restrict__ Qn,
                                                   const double *__restrict__ Kk, double *__restrict__ acc,
                                                   double *__restrict__ Qx, int32_t npatch,
                                                   const int32_t *__restrict__ pface)
{
    constexpr uint32_t WGS = RK4_PARTS + (GHOSTS ? 6 * RK4_CHUNKS : 0);
    constexpr int BATCH = 6;  // slots of an interior cell together
    const uint32_t lb = (uint32_t)xcd_logical_block(blockIdx.x, gridDim.x);
    const int p = (int)(lb / WGS), part = (int)(lb % WGS), i = (int)threadIdx.x;
    if (p >= npatch) return;
    const int64_t leaf = (int64_t)p * PS;
    if (GHOSTS && part >= RK4_PARTS) {
        const int f = (part - RK4_PARTS) / RK4_CHUNKS, first = (part - RK4_PARTS) % RK4_CHUNKS * RK4_CHUNK;
        if (pface[6 * p + f] < 0 || i >= 3 * NFACE) return;
        int L, t1, t2;
        slab_coords(f / 2, i % NFACE, L, t1, t2);
        const int64_t base = leaf + slab_off(f / 2, ghost_c(f % 2 ? 1 : -1, L), t1, t2);
        const int v = first + i / NFACE, end = min(first + RK4_CHUNK, NV);
        rk_combine<(RK4_CHUNK + 2) / 3>(s, dt, Qn, Kk, acc, Qx,
                                        [&](int j) { return v + 3 * j < end ? base + (int64_t)(v + 3 * j) * CS : -1; });
        return;
    }
    if (i >= NCELL) return;
    const int v0 = part == 0 ? 0 : RK4_HEAD + (part - 1) * RK4_REST, v1 = RK4_HEAD + part * RK4_REST;
    const int64_t base = leaf + boff(i % 9 + 3, (i / 9) % 9 + 3, i / 81 + 3);
    if (s < 3 || part > 0) {
        for (int v = v0; v < v1; v += BATCH)
            rk_combine<BATCH>(s, dt, Qn, Kk, acc, Qx,
                              [&](int j) { return v + j < v1 ? base + (int64_t)(v + j) * CS : -1; });
        return;
    }
    double q[RK4_HEAD];
#pragma unroll
    for (int v = 0; v < RK4_HEAD; ++v) {
        const int64_t e = base + (int64_t)v * CS;
        q[v] = acc[e] + (1.0 / 6.0) * dt * Kk[e];
    }
    project_cell(q);
#pragma unroll
    for (int v = 0; v < RK4_HEAD; ++v) Qx[base + (int64_t)v * CS] = q[v];
}

// ------------------------------------------------------------------ constraints
// H = phi^2 gt^ij R_ij + 2/3 K^2 - At_ij At^ij and
// M_i = gt^kl (d_k At_li - Gt^m_li At_km - Gt^m_lk At_im - 3 At_ik P_l/phi) - 2/3 d_i K.
// Only the trace of the Ricci tensor enters.  By the relations of App. B (D for the derivatives of gt,
// P for that of phi, gt^ml gt_jl = delta^m_j)
//   gt^ij R_ij = 2 S - 2 V^l W_l + 2 gt^ij D_i^ml D_jml + Gt^l D_l - gt^ij Gt^l_im Gt^m_lj
//                + 4 (gt^ij d_i P_j - Gt^k P_k) / phi - 6 gt^ij P_i P_j / phi^2,
//   S = (gt^bc gt^ad - gt^ab gt^cd) d_a D_bcd, V^l = D_m^ml, W_l = gt^ij Gt_l,ij, Gt^k = gt^kl W_l,
//   D_l = gt^ij D_lij,
// so that each derivative of D, P, At and K (28 slots) is contracted into one of five numbers as it is
// formed, and nothing of it is kept; phi^2 times the trace is taken, with 1 / phi multiplied out.
//
// One work-group per leaf, one cell per lane: the leaf's nine planes and the four planes and rows at
// distance two that a first difference reaches are staged once (a z-slab each, as the stage kernel
// takes them, stages 60% more lines; and holding all 84 differences needed the whole register file at
// one wave per SIMD; small meshes take slabs all the same, below).  Four slots at a time pass through two buffers, one in flight while the other is
// read.  Bound by the staging: on 16^3 leaves 1.19 -> 0.74 ms (2.26 GB of algorithmic bytes, 0.41 ms at
// the rate of a large read).
namespace cons {
constexpr int ROWS = 13;                    // staged rows of a plane, y = 1..13
constexpr int PITCH = 18, PAIRS = PITCH / 2;  // a row's 16 doubles, the eighth pair repeated
constexpr int PLANE = ROWS * PITCH;
// The staging of a work-group that takes NPL planes of a leaf: its own planes, then the interior rows
// (x = 2..11) of the two planes below and the two above them.
template <int H_ONLY, int NPL>
struct Staging {
    static constexpr int OWN = NPL * PLANE, OWN_PAIRS = NPL * ROWS * PAIRS;
    static constexpr int SLOT = OWN + 4 * PN * LDS_HROW, SLOT_PAIRS = SLOT / 2;
    static constexpr int CELLS = NPL * PN * PN, LANES = (CELLS + 63) / 64 * 64;
    static constexpr int COPIES = (SLOT_PAIRS + LANES - 1) / LANES;  // per lane and slot; the last only of some
    static constexpr int BATCH = H_ONLY ? 3 : (NPL == PN ? 4 : 7);    // slots a round: D and P, or all of them
    static constexpr int ROUNDS = (H_ONLY ? 21 : 28) / BATCH;
    static_assert(BATCH * ROUNDS == (H_ONLY ? 21 : 28) && 2 * BATCH * SLOT * 8 <= 159 * 1024, "staging");
};

// the slot staged as number j: D, P, At, K
__device__ __forceinline__ constexpr int slot(int j)
{
    return j < 18 ? SD + j : (j < 21 ? SP + j - 18 : (j < 27 ? SAT + j - 21 : SK));
}

struct Cell {
    int c, zo[5];    // LDS index of the cell; of its z-neighbours at offset k - 2
    double i12[3];
};

// what the staged slots leave behind
struct Sums {
    double S, Se, trdP, trdPe, M[3], Me[3];  // and what their own roundings took
    double D[3][6], P[3], At[6], K;
};

// s + t into s, the rounding into e.  H is a small difference of S and trdP, whose own roundings are most of
// its error: on gauge waves with a small field in every slot 4.2e-17 rms against an evaluation in extended
// precision, 6.0e-17 with plain sums, 5.2e-17 by way of the Ricci tensor's components (the time is the same).
__device__ __forceinline__ void add(double &s, double &e, double t)
{
    const double r = s + t, u = r - s;
    e += (s - (r - u)) + (t - u);
    s = r;
}
__device__ __forceinline__ double total(double s, double e) { return isfinite(s) ? s + e : s; }
__device__ __forceinline__ constexpr bool cyclic(int i, int j) { return (j - i + 3) % 3 == 1; }

template <int J>
__device__ __forceinline__ void take(const double *__restrict__ f, const Cell &C, const double gd[6], const double ig[6],
                                     Sums &X)
{
    constexpr int v = slot(J);
    const double val = f[C.c];
    double d[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        auto at = [&](int k) { return f[a == 0 ? C.c + k : (a == 1 ? C.c + k * PITCH : C.zo[k + 2])]; };
        d[a] = (8.0 * (at(1) - at(-1)) - (at(2) - at(-2))) * C.i12[a];
    }
    // 0, or NaN where a difference is not finite: such a cell's H is NaN, whichever terms the difference enters
    const double spoiled = 0.0 * (d[0] + d[1] + d[2]);
    if constexpr (v >= SD && v < SP) {
        // the coefficient of d_a D_bcd in S is a 2 x 2 minor of the inverse metric: eps^bdm eps^can gt_mn / det gt
        // (none of D_bbb's differences enters)
        constexpr int b = (v - SD) / 6, s = (v - SD) % 6;
        X.D[b][s] = val;
        double t = spoiled;
#pragma unroll
        for (int o = 0; o < 2; ++o) {  // (c, d) in both orders
            const int c = o ? sym_second(s) : sym_first(s), e = o ? sym_first(s) : sym_second(s);
            if (e == b || (o && c == e)) continue;
#pragma unroll
            for (int a = 0; a < 3; ++a)
                if (a != c) {
                    const double m = gd[sym(3 - b - e, 3 - c - a)];
                    t += (cyclic(b, e) == cyclic(c, a) ? m : -m) * d[a];
                }
        }
        add(X.S, X.Se, t);
    } else if constexpr (v >= SP && v < SK0) {
        constexpr int j = v - SP;
        X.P[j] = val;
        add(X.trdP, X.trdPe, ig[sym(0, j)] * d[0] + ig[sym(1, j)] * d[1] + ig[sym(2, j)] * d[2] + spoiled);
    } else if constexpr (v >= SAT && v < SAT + 6) {
        constexpr int s = v - SAT, l = sym_first(s), i = sym_second(s);
        X.At[s] = val;
        add(X.M[i], X.Me[i], ig[sym(0, l)] * d[0] + ig[sym(1, l)] * d[1] + ig[sym(2, l)] * d[2]);
        if (l != i) add(X.M[l], X.Me[l], ig[sym(0, i)] * d[0] + ig[sym(1, i)] * d[1] + ig[sym(2, i)] * d[2]);
    } else {
        X.K = val;
#pragma unroll
        for (int i = 0; i < 3; ++i) add(X.M[i], X.Me[i], -(2.0 / 3.0) * d[i]);
    }
    // materialised here: the sums are used at the end only, and the compiler would otherwise move their
    // arithmetic there and keep every stencil value until then
    asm volatile("" : "+v"(X.S), "+v"(X.Se), "+v"(X.trdP), "+v"(X.trdPe) : : "memory");
#pragma unroll
    for (int i = 0; i < 3; ++i) asm volatile("" : "+v"(X.M[i]), "+v"(X.Me[i]) : : "memory");
}

// slots J0..J0 + N - 1, each STRIDE doubles after the one before
template <int J0, int N, int STRIDE>
__device__ __forceinline__ void take_all(const double *__restrict__ f, const Cell &C, const double gd[6],
                                         const double ig[6], Sums &X)
{
    take<J0>(f, C, gd, ig, X);
    if constexpr (N > 1) take_all<J0 + 1, N - 1, STRIDE>(f + STRIDE, C, gd, ig, X);
}

// H and M_i (or H only) from the sums, the metric's inverse and phi
template <int H_ONLY>
__device__ __forceinline__ void finish(const Sums &X, const double ig[6], double phi, double hm[4])
{
    auto mult = [](int s) { return s == 0 || s == 3 || s == 5 ? 1.0 : 2.0; };
    const double (&D)[3][6] = X.D;
    double V[3] = {0.0, 0.0, 0.0}, trD[3], W[3], Gv[3], DD = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        double Dm[3][3], Dup[6], t = 0.0;
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int m = 0; m < 3; ++m)
                Dm[i][m] = ig[sym(i, 0)] * D[k][sym(0, m)] + ig[sym(i, 1)] * D[k][sym(1, m)] + ig[sym(i, 2)] * D[k][sym(2, m)];
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = i; j < 3; ++j)
                Dup[sym(i, j)] = Dm[i][0] * ig[sym(0, j)] + Dm[i][1] * ig[sym(1, j)] + Dm[i][2] * ig[sym(2, j)];
#pragma unroll
        for (int l = 0; l < 3; ++l) V[l] += Dup[sym(k, l)];
        trD[k] = Dm[0][0] + Dm[1][1] + Dm[2][2];
#pragma unroll
        for (int s = 0; s < 6; ++s)
            t += mult(s) * Dup[s] * (ig[sym(k, 0)] * D[0][s] + ig[sym(k, 1)] * D[1][s] + ig[sym(k, 2)] * D[2][s]);
        DD += t;
    }
    double Gt[3][6];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = i; j < 3; ++j) {
            double low[3];
#pragma unroll
            for (int l = 0; l < 3; ++l) low[l] = D[i][sym(j, l)] + D[j][sym(i, l)] - D[l][sym(i, j)];
#pragma unroll
            for (int k = 0; k < 3; ++k)
                Gt[k][sym(i, j)] = ig[sym(k, 0)] * low[0] + ig[sym(k, 1)] * low[1] + ig[sym(k, 2)] * low[2];
        }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        Gv[k] = 0.0;
#pragma unroll
        for (int s = 0; s < 6; ++s) Gv[k] += mult(s) * ig[s] * Gt[k][s];
    }
#pragma unroll
    for (int l = 0; l < 3; ++l) {  // W_l = 2 gt^ij D_ijl - D_l
        double t = 0.0;
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) t += ig[sym(i, j)] * D[i][sym(j, l)];
        W[l] = 2.0 * t - trD[l];
    }
    double GG = 0.0;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = i; j < 3; ++j) {
            double t = 0.0;
#pragma unroll
            for (int l = 0; l < 3; ++l)
#pragma unroll
                for (int m = 0; m < 3; ++m) t += Gt[l][sym(i, m)] * Gt[m][sym(l, j)];
            GG += mult(sym(i, j)) * ig[sym(i, j)] * t;
        }
    const double iphi = 1.0 / phi;
    double Pu[3], Am[3][3];
#pragma unroll
    for (int m = 0; m < 3; ++m) Pu[m] = ig[sym(m, 0)] * X.P[0] + ig[sym(m, 1)] * X.P[1] + ig[sym(m, 2)] * X.P[2];
    const double VW = V[0] * W[0] + V[1] * W[1] + V[2] * W[2], GD = Gv[0] * trD[0] + Gv[1] * trD[1] + Gv[2] * trD[2];
    const double GP = Gv[0] * X.P[0] + Gv[1] * X.P[1] + Gv[2] * X.P[2];
    const double PP = X.P[0] * Pu[0] + X.P[1] * Pu[1] + X.P[2] * Pu[2];
    // phi^2 gt^ij R_ij with 1 / phi multiplied out; what has no finite 1 / phi or phi^2 stays marked
    const double R = phi * (phi * (2.0 * (X.S - VW + DD) + (GD - GG)) + 4.0 * (X.trdP - GP)) - 6.0 * PP +
                     0.0 * (iphi + phi * phi);
    double AA = 0.0;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
            Am[i][j] = ig[sym(i, 0)] * X.At[sym(0, j)] + ig[sym(i, 1)] * X.At[sym(1, j)] + ig[sym(i, 2)] * X.At[sym(2, j)];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) AA += Am[i][j] * Am[j][i];
    hm[0] = R + (2.0 / 3.0) * X.K * X.K - AA;
    if (H_ONLY) return;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        double t = X.M[i];
#pragma unroll
        for (int m = 0; m < 3; ++m) {
#pragma unroll
            for (int l = 0; l < 3; ++l) t -= Am[l][m] * Gt[m][sym(l, i)];
            t -= Gv[m] * X.At[sym(i, m)];
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) t -= 3.0 * (Pu[k] * iphi) * X.At[sym(i, k)];
        hm[1 + i] = t;
    }
}
}  // namespace cons

// H_ONLY: what the refinement criterion takes, H of every cell (HM: one value a cell) and nothing else: At
// and K are read pointwise, the slots that are only tested for finiteness not at all, and no norms are
// summed: 4390 lines a leaf instead of 6980.
//
// NPL planes a work-group: the whole leaf, or, while all of a mesh's slabs of three planes run side by side
// (three a leaf on 256 CUs), a slab.  There is then one round of work-groups and its length is the time: a
// third of the LDS reads, seven slots a round instead of four.  See CONS_SLAB_LEAVES.
template <int H_ONLY, int NPL>
__global__ __launch_bounds__((cons::Staging<H_ONLY, NPL>::LANES))
__attribute__((amdgpu_waves_per_eu(NPL / 3, NPL / 3))) void k_constraints_lds(
    const double *__restrict__ Q, double *__restrict__ HM, const PatchGeom *__restrict__ geom, int32_t npatch,
    double r_excise, double *__restrict__ part)
{
    using namespace cons;
    typedef Staging<H_ONLY, NPL> St;
    constexpr int SLOT = St::SLOT, SLOT_PAIRS = St::SLOT_PAIRS, LANES = St::LANES, COPIES = St::COPIES;
    constexpr int BATCH = St::BATCH, ROUNDS = St::ROUNDS;
    __shared__ double bufa[BATCH * SLOT], bufb[BATCH * SLOT];
    __shared__ double red[LANES / 64][4];
    const int lb = (int)xcd_logical_block(blockIdx.x, gridDim.x);
    const int p = lb / (PN / NPL), zb = 3 + NPL * (lb % (PN / NPL));  // the leaf, and the first of the planes
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    double h2 = 0.0, m2 = 0.0, cnt = 0.0, bad = 0.0;
    if (p < npatch) {  // uniform over the work-group
        const PatchBuf qb{Q + (int64_t)p * PS};
        const bool act = tid < St::CELLS;
        const int cc = act ? tid : St::CELLS - 1, m = cc / 9;
        // rows in an order that spreads them over the LDS banks, as slab_row_y, planes of 13 rows
        const int zl = m / 9, k9 = (m + 6 * zl) % 9, yr = k9 / 2 + (k9 % 2 ? 5 : 0), x = cc % 9 + 3;
        const uint32_t ob = 8u * (uint32_t)boff(x, yr + 3, zl + zb);
        // the slots that are only tested, and the metric and phi, first: they are used first
        double g[6], other = 0.0, rest[H_ONLY ? 7 : SAT - 7 + SD - STHETA + 1];
#pragma unroll
        for (int v = 0; v < 6; ++v) g[v] = qb.load(ob, SG + v);
        const double phi = qb.load(ob, SPHI);
        if constexpr (H_ONLY) {
#pragma unroll
            for (int s = 0; s < 7; ++s) rest[s] = qb.load(ob, s < 6 ? SAT + s : SK);
        } else {
            int n = 0;
#pragma unroll
            for (int v = 6; v < SPHI; ++v) rest[n++] = qb.load(ob, v);
#pragma unroll
            for (int v = STHETA; v < SD; ++v) rest[n++] = qb.load(ob, v);
            rest[n++] = qb.load(ob, SK0);
        }
        const double *src[COPIES];
#pragma unroll
        for (int i = 0; i < COPIES; ++i) {
            const int q = min(i * LANES + tid, SLOT_PAIRS - 1);
            int e;
            if (q < St::OWN_PAIRS) {
                const int r = q / PAIRS, j = q % PAIRS;
                e = (zb + r / ROWS) * ZS + (r % ROWS + 1) * XS + 2 * (j < 8 ? j : 7);
            } else {
                const int h = q - St::OWN_PAIRS, hp = h / 45;
                e = (hp < 2 ? zb - 2 + hp : zb + NPL - 2 + hp) * ZS + ((h / 5) % 9 + 3) * YS + 2 + 2 * (h % 5);
            }
            src[i] = qb.base + e;
        }
        const bool last = (COPIES - 1) * LANES + tid < SLOT_PAIRS;
        auto issue = [&](double *buf, int round) {
            double *dst = buf + wave * 128;
#pragma unroll
            for (int j = 0; j < BATCH; ++j)
#pragma unroll
                for (int i = 0; i < COPIES - 1; ++i)
                    __builtin_amdgcn_global_load_lds((const void *)(src[i] + slot(round * BATCH + j) * CS),
                                                     (lds_void_t *)(dst + j * SLOT + i * 2 * LANES), 16, 0, 0);
            if (last)
#pragma unroll
                for (int j = 0; j < BATCH; ++j)
                    __builtin_amdgcn_global_load_lds((const void *)(src[COPIES - 1] + slot(round * BATCH + j) * CS),
                                                     (lds_void_t *)(dst + j * SLOT + (COPIES - 1) * 2 * LANES), 16, 0, 0);
            copies_issued();
        };
        issue(bufa, 0);
        issue(bufb, 1);
        const PatchGeom G = geom[p];
        Cell C;
        C.c = zl * PLANE + (yr + 2) * PITCH + x;
#pragma unroll
        for (int k = -2; k <= 2; ++k) {
            const int z2 = zl + k;
            C.zo[k + 2] = z2 >= 0 && z2 < NPL ? C.c + k * PLANE
                                              : St::OWN + (z2 < 0 ? z2 + 2 : z2 - NPL + 2) * 90 + yr * LDS_HROW + (x - 2);
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) C.i12[a] = 1.0 / (12.0 * G.dx[a]);
        double ig[6], detg;
        metric_inverse(g, ig, detg);
        Sums X;
        if constexpr (H_ONLY) {
#pragma unroll
            for (int s = 0; s < 6; ++s) X.At[s] = rest[s];
            X.K = rest[6];
        } else {
            // 0 times a finite number is 0, anything else is not
#pragma unroll
            for (int v = 0; v < 6; ++v) other += 0.0 * g[v];
#pragma unroll
            for (int n = 0; n < (int)(sizeof(rest) / sizeof(rest[0])); ++n) other += 0.0 * rest[n];
            asm volatile("" : "+v"(other));
        }
        X.S = X.Se = X.trdP = X.trdPe = 0.0;
#pragma unroll
        for (int i = 0; i < 3; ++i) X.M[i] = X.Me[i] = 0.0;
        // the wave's copies of this round have landed (those of the next stay in flight), then those of all waves
        auto wait = [&](bool more) {
            if (!more) wait_memory<0>();
            else if (wave * 64 + (COPIES - 1) * LANES < SLOT_PAIRS) wait_memory<COPIES * BATCH>();
            else wait_memory<(COPIES - 1) * BATCH>();
            lds_swap();
        };
#define CONS_ROUND(R, buf)                                                     \
    if constexpr (R < ROUNDS) {                                                \
        wait(R + 1 < ROUNDS);                                                  \
        take_all<(R < ROUNDS ? R * BATCH : 0), BATCH, SLOT>(buf, C, g, ig, X); \
        if (R + 2 < ROUNDS) {                                                  \
            lds_swap();                                                        \
            issue(buf, R + 2);                                                 \
        }                                                                      \
    }
        CONS_ROUND(0, bufa)
        CONS_ROUND(1, bufb)
        CONS_ROUND(2, bufa)
        CONS_ROUND(3, bufb)
        CONS_ROUND(4, bufa)
        CONS_ROUND(5, bufb)
        CONS_ROUND(6, bufa)
#undef CONS_ROUND
        X.S = total(X.S, X.Se) / detg;
        X.trdP = total(X.trdP, X.trdPe);
#pragma unroll
        for (int i = 0; i < 3; ++i) X.M[i] = total(X.M[i], X.Me[i]);
        double hm[4];
        finish<H_ONLY>(X, ig, phi, hm);
        if constexpr (H_ONLY) {
            if (act) HM[(int64_t)p * NCELL + ((zb - 3 + zl) * 9 + yr) * 9 + x - 3] = hm[0];
        } else if (act) {
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                other += 0.0 * X.P[i];
#pragma unroll
                for (int s = 0; s < 6; ++s) other += 0.0 * X.D[i][s];
            }
#pragma unroll
            for (int s = 0; s < 6; ++s) other += 0.0 * X.At[s];
            other += 0.0 * X.K + 0.0 * phi;
#pragma unroll
            for (int j = 0; j < 4; ++j) other += 0.0 * hm[j];
            const int c = ((zb - 3 + zl) * 9 + yr) * 9 + x - 3;
            if (HM)  // streamed past the caches: the staged lines stay (4096 leaves 724 -> 711 us)
#pragma unroll
                for (int j = 0; j < 4; ++j) __builtin_nontemporal_store(hm[j], HM + ((int64_t)p * 4 + j) * NCELL + c);
            const double X0 = G.org[0] + (x - 2.5) * G.dx[0], Y0 = G.org[1] + (yr + 0.5) * G.dx[1],
                         Z0 = G.org[2] + (zb + zl - 2.5) * G.dx[2];
            const double r = sqrt(X0 * X0 + Y0 * Y0 + Z0 * Z0);
            if (!(other == 0.0)) bad = 1.0;
            else if (r >= r_excise) {
                h2 = hm[0] * hm[0];
                m2 = hm[1] * hm[1] + hm[2] * hm[2] + hm[3] * hm[3];
                cnt = 1.0;
            }
        }
    }
    if (H_ONLY) return;
    // the work-group's sums, in a fixed order: lanes, then waves
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) {
        h2 += __shfl_down(h2, s);
        m2 += __shfl_down(m2, s);
        cnt += __shfl_down(cnt, s);
        bad += __shfl_down(bad, s);
    }
    if ((tid & 63) == 0) {
        red[wave][0] = h2;
        red[wave][1] = m2;
        red[wave][2] = cnt;
        red[wave][3] = bad;
    }
    __syncthreads();
    if (tid < 4) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < LANES / 64; ++w) t += red[w][tid];
        part[(int64_t)blockIdx.x * 4 + tid] = t;
    }
}

// The norms from the work-groups' sums (four numbers each): one work-group, every lane a strided share
// with eight rows in flight, then a tree; in a fixed order.
__global__ __launch_bounds__(1024) void k_reduce_parts(const double *__restrict__ part, int64_t nblk,
                                                       double *__restrict__ out)
{
    __shared__ double red[16][4];
    double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
    for (int64_t b = threadIdx.x; b < nblk; b += 1024)
#pragma unroll
        for (int j = 0; j < 4; ++j) s[j] += part[b * 4 + j];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1)
#pragma unroll
        for (int j = 0; j < 4; ++j) s[j] += __shfl_down(s[j], d);
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int j = 0; j < 4; ++j) red[threadIdx.x >> 6][j] = s[j];
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 1; w < 16; ++w)
#pragma unroll
            for (int j = 0; j < 4; ++j) red[0][j] += red[w][j];
        const double n = red[0][2];
        out[0] = n > 0 ? sqrt(red[0][0] / n) : 0.0;
        out[1] = n > 0 ? sqrt(red[0][1] / n) : 0.0;
        out[2] = red[0][3];
    }
}

// ------------------------------------------------------------------ refinement tags
// one block (256 threads) per leaf; H: one value a cell
__global__ void k_tag_indicator(const double *__restrict__ Q, const double *__restrict__ H,
                                const PatchGeom *__restrict__ geom, double *__restrict__ ind)
{
    const int p = blockIdx.x;
    const double *Qp = Q + (int64_t)p * PS;
    double gc = 0.0, ga = 0.0, hm = 0.0;
    for (int c = threadIdx.x; c < NCELL; c += blockDim.x) {
        const int x = c % 9 + 3, y = (c / 9) % 9 + 3, z = c / 81 + 3;
        const int o = boff(x, y, z);
        const double ph = Qp[SPHI * CS + o], al = Qp[SALPHA * CS + o];
        const double chi = ph * ph;
        const int st[3] = {1, YS, ZS};
        const int cc[3] = {x, y, z};
        for (int a = 0; a < 3; ++a) {
            if (cc[a] + 1 >= 12) continue;
            const double ph2 = Qp[SPHI * CS + o + st[a]];
            gc = fmax(gc, fabs(ph2 * ph2 - chi));
            ga = fmax(ga, fabs(Qp[SALPHA * CS + o + st[a]] - al));
        }
        hm = fmax(hm, fabs(H[(int64_t)p * NCELL + c]));
    }
    __shared__ double red[3][256];
    red[0][threadIdx.x] = gc;
    red[1][threadIdx.x] = ga;
    red[2][threadIdx.x] = hm;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int j = 0; j < 3; ++j) red[j][threadIdx.x] = fmax(red[j][threadIdx.x], red[j][threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double dx = geom[p].dx[0];
        ind[3 * p] = red[0][0];
        ind[3 * p + 1] = red[1][0];
        ind[3 * p + 2] = dx * dx * red[2][0];
    }
}

// sib[p*27 + n]: the 27 sibling leaves of leaf p (-1 if a sibling is not a leaf); level-0 leaves
// have no siblings (sib[p*27] = -2)
__global__ void k_tag_decide(const double *__restrict__ ind, const int32_t *__restrict__ sib,
                             const PatchGeom *__restrict__ geom, int32_t npatch, double theta_r,
                             double theta_c, int32_t max_level, int8_t *__restrict__ tags)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= npatch) return;
    auto e_of = [&](int q) { return fmax(fmax(ind[3 * q], ind[3 * q + 1]), ind[3 * q + 2]); };
    const double e = e_of(p);
    const int lev = geom[p].level;
    int8_t tg = 0;
    if (e >= theta_r) tg = lev < max_level ? 1 : 0;
    else if (lev > 0 && e < theta_c) {
        bool ok = true;
        for (int n = 0; n < 27 && ok; ++n) {
            const int s = sib[(int64_t)p * 27 + n];
            if (s < 0 || !(e_of(s) < theta_c)) ok = false;
        }
        tg = ok ? -1 : 0;
    }
    tags[p] = tg;
}

// ------------------------------------------------------------------ regrid transfer
// REGRID_PARTS work-groups per leaf of the new mesh, a run of slots each.  COPY: the whole box.
// PROLONG: at each fine cell centre the tensor product over the axes of linear interpolation on the
// parent's interior (fine index f = 9 o + x across the parent, u = (f + 1/2)/3 - 1/2,
// l = clamp(floor(u), 0, 7), weights 1 - (u - l), u - l), summed in the order dz, dy, dx.  RESTRICT:
// the mean of the 3^3 fine cells.  No contraction, so that the sums round exactly as written.  BLANK:
// the cells outside the interior of the last two kinds are zeroed (the new state was not written yet).
// Bound by memory: a copied box moves at the rate of a large copy (5.3 TB/s with eight 16-byte loads in
// flight a lane).  An interpolated leaf's parent cells, 5^3 of each slot, are staged at once, so that only
// stores remain between the sums.  5680 leaves, 2662 of them copied, 3014 interpolated: 3.1 ms including
// the task table (3.8 ms with the sums reading global memory; zeroing the state, initial data everywhere
// and transfer, as before, took 5.6 ms).
constexpr int REGRID_PARTS = 8, REGRID_SLOTS = (NV + REGRID_PARTS - 1) / REGRID_PARTS;

template <int BLANK>
__global__ __launch_bounds__(256) void k_regrid(const double *__restrict__ Qo, double *__restrict__ Qn,
                                                const RegridTask *__restrict__ tasks, int32_t n)
{
#pragma clang fp contract(off)
    const int p = (int)(blockIdx.x / REGRID_PARTS);
    if (p >= n) return;
    const int v0 = (int)(blockIdx.x % REGRID_PARTS) * REGRID_SLOTS, nv = min(REGRID_SLOTS, NV - v0);
    const RegridTask &tk = tasks[p];
    const int kind = tk.kind;
    double *dst = Qn + (int64_t)p * PS + (int64_t)v0 * CS;
    if (kind == RG_COPY) {
        typedef double pair __attribute__((ext_vector_type(2), aligned(8)));
        const pair *src = (const pair *)(Qo + (int64_t)tk.src * PS + (int64_t)v0 * CS);
        pair *to = (pair *)dst;
        constexpr int U = 8;
        const int m = nv * (CS / 2);
        for (int e = (int)threadIdx.x; e < m; e += U * 256) {
            pair r[U];
#pragma unroll
            for (int k = 0; k < U; ++k)
                if (e + 256 * k < m) r[k] = src[e + 256 * k];
#pragma unroll
            for (int k = 0; k < U; ++k)
                if (e + 256 * k < m) to[e + 256 * k] = r[k];
        }
        return;
    }
    // the parent's 5^3 cells under the leaf, of all slots
    __shared__ double sm[REGRID_SLOTS * 125];
    if (kind == RG_PROLONG) {
        const double *src = Qo + (int64_t)tk.src * PS + (int64_t)v0 * CS +
                            boff(2 * tk.o[0] + 3, 2 * tk.o[1] + 3, 2 * tk.o[2] + 3);
        for (int e = (int)threadIdx.x; e < nv * 125; e += 256)
            sm[e] = src[(e / 125) * CS + boff(e % 5, (e / 5) % 5, (e / 25) % 5)];
    }
    __syncthreads();
    // blank: whole lines of the box are written, interior and zeros together
    for (int c = (int)threadIdx.x; c < (BLANK ? CS : NCELL); c += 256) {
        const int x = BLANK ? c % XS - 3 : c % 9, y = BLANK ? (c / YS) % NBX - 3 : (c / 9) % 9,
                  z = BLANK ? c / ZS - 3 : c / 81;
        double *d = dst + boff(x + 3, y + 3, z + 3);
        if (BLANK && ((unsigned)x >= 9u || (unsigned)y >= 9u || (unsigned)z >= 9u)) {
            for (int v = 0; v < nv; ++v) d[v * CS] = 0.0;
            continue;
        }
        if (kind == RG_PROLONG) {
            const int fc[3] = {x, y, z};
            int l[3];
            double wt[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const int f = 9 * tk.o[a] + fc[a];
                const double uu = (f + 0.5) / 3.0 - 0.5;
                int ll = (int)floor(uu);
                ll = ll < 0 ? 0 : (ll > PN - 2 ? PN - 2 : ll);
                l[a] = ll - 2 * tk.o[a];  // 0..3
                wt[a] = uu - ll;
            }
            const double *src = sm + l[2] * 25 + l[1] * 5 + l[0];
#pragma unroll 4
            for (int v = 0; v < nv; ++v) {
                double s = 0.0;
#pragma unroll
                for (int dz = 0; dz < 2; ++dz)
#pragma unroll
                    for (int dy = 0; dy < 2; ++dy)
#pragma unroll
                        for (int dx = 0; dx < 2; ++dx) {
                            const double wgt = (dz ? wt[2] : 1.0 - wt[2]) * (dy ? wt[1] : 1.0 - wt[1]) *
                                               (dx ? wt[0] : 1.0 - wt[0]);
                            s += wgt * src[v * 125 + dz * 25 + dy * 5 + dx];
                        }
                d[v * CS] = s;
            }
        } else {
            const int kid = tk.kid[(z / 3) * 9 + (y / 3) * 3 + x / 3];
            const double *src = Qo + (int64_t)kid * PS + (int64_t)v0 * CS +
                                boff(3 * (x % 3) + 3, 3 * (y % 3) + 3, 3 * (z % 3) + 3);
            for (int v = 0; v < nv; ++v) {
                double s = 0.0;
#pragma unroll
                for (int dz = 0; dz < 3; ++dz)
#pragma unroll
                    for (int dy = 0; dy < 3; ++dy)
#pragma unroll
                        for (int dx = 0; dx < 3; ++dx) s += src[v * CS + boff(dx, dy, dz)];
                d[v * CS] = s / 27.0;
            }
        }
    }
}

// Differences of primaries V0..V1-1, staged in LDS buffers 0.., into the auxiliaries of the cell.
template <int V0, int V1, int XG>
__device__ __forceinline__ void reconstruct_from_lds(const LdsCell<XG> &C, double *__restrict__ qb, int o,
                                                     const int64_t (&pd)[3], int rest)
{
#pragma unroll
    for (int v = V0; v < V1; ++v)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const double d = fd(C, v - V0, a);
            // D_a(ij) = d_a gt_ij / 2, A_a = d_a alpha, B_a^i = d_a beta^i, P_a = d_a phi
            const int dst = v < SALPHA ? SD + 6 * a + v
                          : v == SALPHA ? SA + a
                          : v < SPHI ? SB + 3 * a + (v - SBETA)
                                     : SP + a;
            const double u = v < SALPHA ? 0.5 * d : d;
            const int64_t e = (int64_t)dst * CS + o;
            qb[e] = u;
            if (rest != 0) qb[e + rest] = u;
            if (pd[0] != 0) qb[e + pd[0]] = u;
#pragma unroll
            for (int k = 1; k < 3; ++k)  // streamed, as the stage sink's y and z copies
                if (pd[k] != 0) __builtin_nontemporal_store(u, qb + e + pd[k]);
        }
}

// Second-order formulation (Sec. 3.2, explicit gradient reconstruction; Algorithm 2): the
// auxiliaries from central FD4 differences of the primaries by their definitions,
// A_k = d_k alpha, B_k^i = d_k beta^i, D_kij = d_k gt_ij / 2, P_k = d_k phi, on the interior
// cells of every leaf.  One work-group per z-slab copies the slab's 11 primaries into LDS exactly as
// the stage kernel stages a slot (the slab's planes with their x and y halos, the interior rows of
// the three planes below and above), then every lane forms its cell's 33 differences from LDS
// (116 KiB: one work-group per CU; two rounds of six primaries in 63 KiB, two work-groups per CU, ran
// 5% slower; one thread per cell reading its stencils through the caches ran 30% slower).  The
// primaries' halos must be filled, except the face halos normal to an axis of gaxes and shared with a
// same-level leaf, which are read from that leaf's interior.  Every value within
// three layers of a face shared with a same-level leaf and normal to an axis of paxes is also
// written into that leaf's face halo (as the stage push does).  Inside a step (XG, no copies) whole rows
// are written (row_rest): a step of the second-order formulation on 16^3 leaves 17.43 -> 17.18 ms.
// The lanes take the slab's rows in their natural order, not in that of slab_row_y: the stores bound it, not
// the LDS, and a wave then writes the rows of a neighbour's halo side by side (4096 leaves with copies 1.70 ms,
// 1.75 ms in that order; without copies 0.77 ms in both).
template <int XG>
__global__ __launch_bounds__(256) void k_reconstruct_lds(double *__restrict__ Q, const PatchGeom *__restrict__ geom,
                                                         int32_t npatch, const int32_t *__restrict__ nbr,
                                                         int32_t paxes, int32_t gaxes,
                                                         const int32_t *__restrict__ pface)
{
    __shared__ double lds[LDS_A], ldsb[(SPHI + 1 - LDS_NA) * LDS_SLOT];
    const int64_t lb = xcd_logical_block(blockIdx.x, gridDim.x);
    const int p = (int)(lb / 3);
    if (p >= npatch) return;  // uniform over the work-group
    const int sl = (int)(lb % 3);
    const PatchGeom g = geom[p];
    const bool act = (int)threadIdx.x < NFACE;
    const int cc = act ? (int)threadIdx.x : NFACE - 1, x = cc % 9 + 3, y = (cc / 9) % 9 + 3, zl = cc / 81;
    const HaloSrc hs = halo_sources(nbr, p, gaxes);
    LdsCell<XG> C;
    C.s = lds;
    C.sb = ldsb;
    lds_cell_offsets(C, x, y, zl, hs);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        C.i12[a] = 1.0 / (12.0 * g.dx[a]);
        C.koc[a] = 0.0;
    }
    double *qb = Q + (int64_t)p * PS;
    const int z = zl + 3 + 3 * sl;
    const int o = boff(x, y, z);
    int64_t pd[3];
    push_offsets(paxes ? nbr : nullptr, p, x, y, z, o, pd, paxes);
    const int slots[LDS_NA] = {0, 1, 2, 3, 4, 5, 6, 7, 8}, slotsb[SPHI + 1 - LDS_NA] = {9, 10};
    const Stager sg = lds_stager<XG>(qb, sl, hs);
    lds_issue(lds, slots, sg);
    lds_issue(ldsb, slotsb, sg);
    wait_memory<0>();
    lds_swap();
    if (act) reconstruct_from_lds<0, SPHI + 1, XG>(C, qb, o, pd, XG && !paxes ? row_rest(x, pface, p) : 0);
}


hipError_t launch_reconstruct(double *Q, const PatchGeom *geom, int32_t npatch, const int32_t *nbr, int32_t paxes,
                              int32_t gaxes, const int32_t *pface, hipStream_t st)
{
    if (npatch <= 0) return hipSuccess;
    const int64_t nb = ((int64_t)npatch * 3 + 7) / 8 * 8;  // a multiple of 8 for the XCD block order
    if (gaxes & 1)
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_reconstruct_lds<1>), dim3((unsigned)nb), dim3(256), 0, st, Q, geom, npatch,
                           nbr, paxes, gaxes, pface);
    else
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_reconstruct_lds<0>), dim3((unsigned)nb), dim3(256), 0, st, Q, geom, npatch,
                           nbr, paxes, gaxes, pface);
    return hipGetLastError();
}

// The cube index of coordinate v at the finest level, and whether leaf g (level l, lower corner
// org + i * edge_l) holds that index: i * 3^(top - l) <= K < (i + 1) * 3^(top - l).  One rounded
// index serves every level, so the leaves tile the domain without gaps or overlaps even for points
// within rounding of a face.
__device__ __forceinline__ double fine_index(const LeafLookup &lk, int a, double v)
{
    return floor((v - lk.org[a]) / lk.fine[a]);
}
__device__ __forceinline__ bool leaf_holds(const LeafLookup &lk, const PatchGeom &g, const double K[3])
{
    double s = 1.0;
    for (int l = g.level; l < lk.top; ++l) s *= 3.0;
    bool in = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double i = rint((g.org[a] - lk.org[a]) / (lk.fine[a] * s));
        in = in && K[a] >= i * s && K[a] < (i + 1.0) * s;
    }
    return in;
}

// Tracers (Sec. 3.8): one work-group per point.  The lanes test a strided share of the leaves for
// the one holding the point (leaf_holds); the trilinear weights come from the 2^3 cell centres
// around the point at that leaf's spacing.  A cell inside the leaf's interior is read there; a
// cell outside it is read from the interior of the leaf of the same level that holds its centre
// (a second strided search), so that no value comes from an edge or corner region of a halo,
// which no fill writes; a cell whose centre is outside the domain or in a leaf of another level is
// read from the leaf's own box (its face halo, filled by the boundary or coarse-fine fill).  Each
// requested slot is then interpolated by one lane.  advance: the point moves by dt * (-beta)
// (puncture tracker, explicit Euler).  A point outside every leaf samples NaN and stays.
__global__ __launch_bounds__(256) void k_tracers(const double *__restrict__ Q, const PatchGeom *__restrict__ geom,
                                                 int32_t npatch, double *__restrict__ pos, TracerSlots sl,
                                                 LeafLookup lk, double *__restrict__ out, double dt,
                                                 int32_t advance)
{
    __shared__ int leaf;
    __shared__ int owner[8];
    __shared__ double beta[3];
    const int64_t i = blockIdx.x;
    if (threadIdx.x == 0) leaf = -1;
    if (threadIdx.x < 8) owner[threadIdx.x] = -1;
    __syncthreads();
    const double x[3] = {pos[3 * i], pos[3 * i + 1], pos[3 * i + 2]};
    const double K[3] = {fine_index(lk, 0, x[0]), fine_index(lk, 1, x[1]), fine_index(lk, 2, x[2])};
    for (int p = (int)threadIdx.x; p < npatch; p += (int)blockDim.x)
        if (leaf_holds(lk, geom[p], K)) leaf = p;  // one leaf holds a point: one lane at most
    __syncthreads();
    const int p = leaf;  // uniform over the work-group
    int i0[3] = {3, 3, 3};
    double w[3] = {0.0, 0.0, 0.0};
    PatchGeom gp{};
    if (p >= 0) {
        gp = geom[p];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const double u = (x[a] - gp.org[a]) / gp.dx[a] - 0.5;
            const double f = floor(u);
            i0[a] = (int)f + 3;  // box index of the lower centre: 2..11
            w[a] = u - f;
        }
        // owners of the cells outside the leaf's interior (one leaf holds a centre: one lane each)
        for (int q = (int)threadIdx.x; q < npatch; q += (int)blockDim.x) {
            const PatchGeom g = geom[q];
            if (q == p || g.level != gp.level) continue;
            for (int c = 0; c < 8; ++c) {
                const int b[3] = {i0[0] + (c & 1), i0[1] + ((c >> 1) & 1), i0[2] + ((c >> 2) & 1)};
                if (b[0] >= 3 && b[0] <= 11 && b[1] >= 3 && b[1] <= 11 && b[2] >= 3 && b[2] <= 11) continue;
                double Kc[3];
#pragma unroll
                for (int a = 0; a < 3; ++a)
                    Kc[a] = fine_index(lk, a, gp.org[a] + ((double)(b[a] - 3) + 0.5) * gp.dx[a]);
                if (leaf_holds(lk, g, Kc)) owner[c] = q;
            }
        }
    }
    __syncthreads();
    const int nout = advance ? 3 : sl.n;
    const int t = (int)threadIdx.x;
    if (t < nout) {
        const int v = advance ? SBETA + t : sl.v[t];
        double val = __builtin_nan("");
        if (p >= 0) {
            val = 0.0;
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const int cx = c & 1, cy = (c >> 1) & 1, cz = (c >> 2) & 1;
                int b[3] = {i0[0] + cx, i0[1] + cy, i0[2] + cz};
                int q = owner[c];
                if (q >= 0) {
                    const PatchGeom g = geom[q];
#pragma unroll
                    for (int a = 0; a < 3; ++a) {
                        const double xc = gp.org[a] + ((double)(b[a] - 3) + 0.5) * gp.dx[a];
                        b[a] = min(11, max(3, (int)floor((xc - g.org[a]) / g.dx[a]) + 3));
                    }
                } else {
                    q = p;
                }
                const double wt = (cx ? w[0] : 1.0 - w[0]) * (cy ? w[1] : 1.0 - w[1]) * (cz ? w[2] : 1.0 - w[2]);
                val += wt * Q[(int64_t)q * PS + v * CS + boff(b[0], b[1], b[2])];
            }
        }
        if (advance) beta[t] = val;
        else out[i * sl.n + t] = val;
    }
    if (advance) {
        __syncthreads();
        if (t == 0 && p >= 0)
#pragma unroll
            for (int a = 0; a < 3; ++a) pos[3 * i + a] = x[a] + dt * (-beta[a]);
    }
}

hipError_t launch_tracers(const double *Q, const PatchGeom *geom, int32_t npatch, int64_t n, double *pos,
                          const TracerSlots &sl, const LeafLookup &lk, double *out, double dt, int32_t advance, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_tracers, dim3((unsigned)n), dim3(256), 0, st, Q, geom, npatch, pos, sl, lk, out, dt, advance);
    return hipGetLastError();
}

// Tracker-based refinement (refinement by coordinates): REFINE a leaf of level l < min(max_level,
// radii.n) whose closed cube lies within r[l] of a tracer; COARSEN a leaf of level >= 1 whose parent
// cube lies farther than r[l - 1] from every tracer; KEEP otherwise.  One lane per leaf.
__device__ __forceinline__ double cube_distance(const double lo[3], const double L[3], int64_t n,
                                                const double *__restrict__ pos)
{
    double best = __builtin_huge_val();
    for (int64_t i = 0; i < n; ++i) {
        double d2 = 0.0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const double x = pos[3 * i + a];
            const double c = x < lo[a] ? lo[a] : (x > lo[a] + L[a] ? lo[a] + L[a] : x);
            d2 += (c - x) * (c - x);
        }
        best = fmin(best, sqrt(d2));
    }
    return best;
}

__global__ __launch_bounds__(256) void k_tag_tracers(const TrackBox *__restrict__ box, int32_t npatch, int64_t n,
                                                     const double *__restrict__ pos, TrackRadii R, int32_t max_level,
                                                     int8_t *__restrict__ tags)
{
    const int p = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (p >= npatch) return;
    const TrackBox b = box[p];
    int8_t t = 0;
    if (b.level < max_level && b.level < R.n && cube_distance(b.lo, b.L, n, pos) <= R.r[b.level])
        t = 1;
    else if (b.level >= 1 && (b.level - 1 >= R.n || cube_distance(b.plo, b.pL, n, pos) > R.r[b.level - 1]))
        t = -1;
    tags[p] = t;
}

hipError_t launch_tag_tracers(const TrackBox *box, int32_t npatch, int64_t n, const double *pos, const TrackRadii &R,
                              int32_t max_level, int8_t *tags, hipStream_t st)
{
    if (npatch <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_tag_tracers, dim3((unsigned)((npatch + 255) / 256)), dim3(256), 0, st, box, npatch, n, pos, R,
                       max_level, tags);
    return hipGetLastError();
}

hipError_t launch_regrid(const double *Qo, double *Qn, const RegridTask *tasks, int32_t n, int32_t blank, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const dim3 g((unsigned)n * REGRID_PARTS);
    if (blank) hipLaunchKernelGGL(HIP_KERNEL_NAME(k_regrid<1>), g, dim3(256), 0, st, Qo, Qn, tasks, n);
    else hipLaunchKernelGGL(HIP_KERNEL_NAME(k_regrid<0>), g, dim3(256), 0, st, Qo, Qn, tasks, n);
    return hipGetLastError();
}

// ------------------------------------------------------------------ launchers
hipError_t launch_init(double *Q, const PatchGeom *geom, int32_t npatch, int32_t scen, const InitArgs &a, hipStream_t st)
{
    const int64_t n = (int64_t)npatch * NCELL;
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_init, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, Q, geom, npatch, scen, a);
    return hipGetLastError();
}

hipError_t launch_init_ghosts(double *Q, const PatchGeom *geom, const BoundaryFace *bf, double *bg, int32_t nbf,
                              const RegridTask *tasks, int32_t scen, const InitArgs &a, hipStream_t st)
{
    if (nbf <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_init_ghosts, dim3(nbf), dim3(256), 0, st, Q, geom, bf, bg, nbf, tasks, scen, a);
    return hipGetLastError();
}

hipError_t launch_fill(double *Q, const FaceTask *tasks, int32_t ntask, int32_t transfer, int32_t v0, int32_t v1,
                       hipStream_t st)
{
    if (ntask <= 0 || v1 <= v0) return hipSuccess;
    const unsigned batches = (unsigned)((v1 - v0 + FILL_SLOTS - 1) / FILL_SLOTS);
    if (transfer == 1)
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_fill<1>), dim3(ntask, batches), dim3(256), 0, st, Q, tasks,
                           ntask, v0, v1);
    else
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_fill<0>), dim3(ntask, batches), dim3(256), 0, st, Q, tasks,
                           ntask, v0, v1);
    return hipGetLastError();
}

hipError_t launch_copy_faces(double *Q, const int32_t *nbr, int32_t npatch, hipStream_t st)
{
    if (npatch <= 0) return hipSuccess;
    const int64_t nb = ((int64_t)npatch + 7) / 8 * 8 * COPY_BATCHES;  // a multiple of 8 for the XCD block order
    hipLaunchKernelGGL(k_copy_faces, dim3((unsigned)nb), dim3(COPY_LANES), 0, st, Q, nbr, npatch);
    return hipGetLastError();
}

hipError_t launch_rhs(const double *Q, double *K, const PatchGeom *geom, int32_t npatch, const RhsParams &p,
                      int32_t precision, int32_t variant, const int32_t *order, const BoundaryFace *bf,
                      const double *bg, int32_t nbf, const int32_t *pface, hipStream_t st)
{
    // the LDS kernel computes the Sommerfeld ghosts' right-hand side inside the slab work-groups;
    // the phased kernel leaves it to k_rhs_sommerfeld
    const int32_t *slab_ghosts = nbf > 0 ? pface : nullptr;
    const int64_t nb = ((int64_t)npatch * 3 + 7) / 8 * 8;
    const int32_t lin = (variant & KV_LINEAR) ? 1 : 0;
    if (variant & KV_LDS) {
        const RhsLaunch a{Q, K, geom, npatch, p, bf, bg, slab_ghosts, lin, order, (int32_t)nb};
        if (p.advection) return precision == 1 ? launch_rhs_lds<float, 1>(a, st) : launch_rhs_lds<double, 1>(a, st);
        return precision == 1 ? launch_rhs_lds<float, 0>(a, st) : launch_rhs_lds<double, 0>(a, st);
    } else {
        const dim3 g((unsigned)nb), b(256);
        if (p.advection) {
            if (precision == 1)
                hipLaunchKernelGGL(HIP_KERNEL_NAME(k_rhs<float, 1>), g, b, 0, st, Q, K, geom, npatch, p, lin, order);
            else
                hipLaunchKernelGGL(HIP_KERNEL_NAME(k_rhs<double, 1>), g, b, 0, st, Q, K, geom, npatch, p, lin, order);
        } else {
            if (precision == 1)
                hipLaunchKernelGGL(HIP_KERNEL_NAME(k_rhs<float, 0>), g, b, 0, st, Q, K, geom, npatch, p, lin, order);
            else
                hipLaunchKernelGGL(HIP_KERNEL_NAME(k_rhs<double, 0>), g, b, 0, st, Q, K, geom, npatch, p, lin, order);
        }
        if (nbf > 0) {
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
            return launch_rhs_sommerfeld(Q, K, geom, bf, bg, nbf, p.shift == 0 ? 1 : 0, st);
        }
    }
    return hipGetLastError();
}

// 3 work-groups per patch (grid padded to a multiple of 8 for the XCD mapping).  The Sommerfeld
// ghost faces get one more work-group each in the same launch with the phased kernel; with the
// LDS kernel each slab work-group updates the ghost cells beside its own planes.
hipError_t launch_stage(int32_t s, double dt, const double *Qs, const double *Qn, double *acc, double *Qx,
                        const PatchGeom *geom, int32_t npatch, const RhsParams &p, int32_t precision,
                        int32_t variant, const int32_t *order, const BoundaryFace *bf, const double *bg, int32_t nbf,
                        const int32_t *pface, const int32_t *nbr, int32_t paxes, int32_t gaxes, int32_t closed,
                        hipStream_t st)
{
    // the LDS kernel updates the Sommerfeld ghosts inside the slab work-groups (per-leaf face table)
    const int32_t *slab_ghosts = nbf > 0 ? pface : nullptr;
    const int64_t nb_slab = ((int64_t)npatch * 3 + 7) / 8 * 8;
    const int64_t nb = nb_slab + (nbf > 0 ? nbf : 0);
    const int32_t ns = (int32_t)nb_slab;
    const int32_t lin = (variant & KV_LINEAR) ? 1 : 0;
    const int32_t *pushed = paxes ? nbr : nullptr;
    if (variant & KV_LDS) {
        const StageLaunch a{Qs, Qn, acc, Qx, geom, npatch, p, s, dt, bf, bg, slab_ghosts, nbr, paxes, gaxes, closed, lin,
                            order, ns};
        if (p.advection) return precision == 1 ? launch_stage_lds<float, 1>(a, st) : launch_stage_lds<double, 1>(a, st);
        return precision == 1 ? launch_stage_lds<float, 0>(a, st) : launch_stage_lds<double, 0>(a, st);
    } else {
        const dim3 g((unsigned)nb), b(256);
        if (p.advection) {
            if (precision == 1)
                hipLaunchKernelGGL(HIP_KERNEL_NAME(k_stage<float, 1>), g, b, 0, st, Qs, Qn, acc, Qx, geom, npatch, ns,
                                   p, s, dt, bf, bg, pushed, paxes, lin, order);
            else
                hipLaunchKernelGGL(HIP_KERNEL_NAME(k_stage<double, 1>), g, b, 0, st, Qs, Qn, acc, Qx, geom, npatch, ns,
                                   p, s, dt, bf, bg, pushed, paxes, lin, order);
        } else {
            if (precision == 1)
                hipLaunchKernelGGL(HIP_KERNEL_NAME(k_stage<float, 0>), g, b, 0, st, Qs, Qn, acc, Qx, geom, npatch, ns,
                                   p, s, dt, bf, bg, pushed, paxes, lin, order);
            else
                hipLaunchKernelGGL(HIP_KERNEL_NAME(k_stage<double, 0>), g, b, 0, st, Qs, Qn, acc, Qx, geom, npatch, ns,
                                   p, s, dt, bf, bg, pushed, paxes, lin, order);
        }
    }
    return hipGetLastError();
}

hipError_t launch_rhs_sommerfeld(const double *Q, double *K, const PatchGeom *geom, const BoundaryFace *bf,
                                 const double *bg, int32_t nbf, int32_t frozen, hipStream_t st)
{
    if (nbf <= 0) return hipSuccess;
    const int64_t n = (int64_t)nbf * NV * NFACE;
    hipLaunchKernelGGL(k_rhs_sommerfeld, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, Q, K, geom, bf, bg,
                       nbf, frozen);
    return hipGetLastError();
}

hipError_t launch_capture_bg(const double *Q, const BoundaryFace *bf, double *bg, int32_t nbf, hipStream_t st)
{
    if (nbf <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_capture_bg, dim3(nbf), dim3(256), 0, st, Q, bf, bg, nbf);
    return hipGetLastError();
}

hipError_t launch_rk4(int32_t s, double dt, const double *Qn, const double *K, double *acc, double *Qx,
                      int32_t npatch, const int32_t *pface, hipStream_t st)
{
    if (npatch <= 0) return hipSuccess;
    const unsigned n8 = ((unsigned)npatch + 7) / 8 * 8;  // a multiple of 8 for the XCD block order
    auto go = [&](auto kernel, unsigned per_leaf) {
        hipLaunchKernelGGL(kernel, dim3(n8 * per_leaf), dim3(RK4_LANES), 0, st, s, dt, Qn, K, acc, Qx, npatch, pface);
    };
    if (pface) go(k_rk4<1>, RK4_PARTS + 6 * RK4_CHUNKS);
    else go(k_rk4<0>, RK4_PARTS);
    return hipGetLastError();
}

// One work-group per leaf, or three where the slabs of all leaves run at once; a multiple of 8 for the XCD
// block order (at least 8).  The line: 256 CUs, one work-group each.  H and M of 1 / 27 / 64 / 85 leaves by
// leaves 28 / 30 / 31 / 32 us, by slabs 16 / 17 / 20 / 22 us, and 32 us by leaves just above it.
constexpr int32_t CONS_SLAB_LEAVES = 256 / 3;
static int64_t blocks_of(int64_t n) { return std::max<int64_t>(8, (n + 7) / 8 * 8); }
int64_t constraints_blocks(int32_t npatch) { return blocks_of(npatch <= CONS_SLAB_LEAVES ? 3 * (int64_t)npatch : npatch); }

hipError_t launch_constraints(const double *Q, double *HM, const PatchGeom *geom, int32_t npatch,
                              double r_excise, double *part, double *out3, hipStream_t st)
{
    const int64_t nb = constraints_blocks(npatch);
    if (npatch <= CONS_SLAB_LEAVES)
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_constraints_lds<0, 3>), dim3((unsigned)nb),
                           dim3(cons::Staging<0, 3>::LANES), 0, st, Q, HM, geom, npatch, r_excise, part);
    else
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_constraints_lds<0, PN>), dim3((unsigned)nb),
                           dim3(cons::Staging<0, PN>::LANES), 0, st, Q, HM, geom, npatch, r_excise, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_reduce_parts, dim3(1), dim3(1024), 0, st, part, nb, out3);
    return hipGetLastError();
}

hipError_t launch_tags(const double *Q, double *H, const PatchGeom *geom, const int32_t *sib,
                       int32_t npatch, double theta_r, double theta_c, int32_t max_level, int8_t *tags,
                       double *ind, hipStream_t st)
{
    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_constraints_lds<1, PN>), dim3((unsigned)blocks_of(npatch)),
                       dim3(cons::Staging<1, PN>::LANES), 0, st, Q, H, geom, npatch, 0.0, nullptr);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_tag_indicator, dim3(npatch), dim3(256), 0, st, Q, H, geom, ind);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_tag_decide, dim3((npatch + 127) / 128), dim3(128), 0, st, ind, sib, geom, npatch,
                       theta_r, theta_c, max_level, tags);
    return hipGetLastError();
}

}  // namespace ccz4
