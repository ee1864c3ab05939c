// Device helpers shared by the kernels' translation units: face-slab coordinates, block order, halo
// copies, the algebraic projection and the Sommerfeld ghost cells.
#pragma once
#include "ccz4_algebra.hpp"

namespace ccz4 {

constexpr int SB8 = 8;  // slots per batch of loads

// det gt = 1 by rescaling, then remove the trace of At with the rescaled metric
__device__ inline void project_cell(double *q)
{
    const double det = q[0] * (q[3] * q[5] - q[4] * q[4]) - q[1] * (q[1] * q[5] - q[4] * q[2]) +
                       q[2] * (q[1] * q[4] - q[3] * q[2]);
    const double s = 1.0 / cbrt(det);
    double g[6];
    for (int v = 0; v < 6; ++v) g[v] = q[v] * s;
    const double c00 = g[3] * g[5] - g[4] * g[4], c01 = g[2] * g[4] - g[1] * g[5], c02 = g[1] * g[4] - g[2] * g[3];
    const double c11 = g[0] * g[5] - g[2] * g[2], c12 = g[1] * g[2] - g[0] * g[4], c22 = g[0] * g[3] - g[1] * g[1];
    const double dn = g[0] * c00 + g[1] * c01 + g[2] * c02;
    const double tr = (c00 * q[11] + c11 * q[14] + c22 * q[16] + 2.0 * (c01 * q[12] + c02 * q[13] + c12 * q[15])) / dn;
    for (int v = 0; v < 6; ++v) {
        q[v] = g[v];
        q[11 + v] -= g[v] * tr * (1.0 / 3.0);
    }
}

// Axis a face: ghost layer L (1..3) sits at box coordinate 11 + L (side +1) or 3 - L (side -1);
// interior depth d (1..3) from the face at 12 - d (side +1) or 2 + d (side -1).
__device__ __forceinline__ int ghost_c(int side, int L) { return side > 0 ? 11 + L : 3 - L; }
__device__ __forceinline__ int depth_c(int side, int d) { return side > 0 ? 12 - d : 2 + d; }

// slab thread -> (layer L in 1..3, tangential t1, t2 in 0..8) with the lowest box axis fastest
__device__ __forceinline__ void slab_coords(int axis, int idx, int &L, int &t1, int &t2)
{
    if (axis == 0) {  // layer index is the contiguous x
        L = idx % 3 + 1;
        t1 = (idx / 3) % 9;   // y
        t2 = idx / 27;        // z
    } else {
        t1 = idx % 9;         // x
        t2 = (idx / 9) % 9;   // z (axis 1) or y (axis 2)
        L = idx / 81 + 1;
    }
}

__device__ __forceinline__ int slab_off(int axis, int coordA, int t1, int t2)
{
    // t1/t2 are the tangential axes in increasing order: axis0 -> (y, z); axis1 -> (x, z); axis2 -> (x, y)
    if (axis == 0) return boff(coordA, t1 + 3, t2 + 3);
    if (axis == 1) return boff(t1 + 3, coordA, t2 + 3);
    return boff(t1 + 3, t2 + 3, coordA);
}

__device__ __forceinline__ bool frozen_slot(int v)
{
    return (v >= SBETA && v < SBETA + 3) || (v >= SBB && v < SBB + 3) || (v >= SB && v < SB + 9);
}

// Work-group -> (patch, z-slab of 3 planes) with the three slabs of a patch on one XCD:
// consecutive block ids are dealt to the 8 XCDs in turn, so logical block L runs at physical
// id (L % per) * 8 + L / per with per = grid / 8 (the grid is padded to a multiple of 8).
__device__ __forceinline__ int64_t xcd_logical_block(int64_t b, int64_t nblk)
{
    const int64_t per = nblk / 8;
    return (b % 8) * per + b / 8;
}

// Offsets (in doubles, relative to the cell's own element) of the copies of interior cell
// (x, y, z) of patch p in the face halos of its same-level neighbours: a cell within three layers
// of a face whose neighbour nbr[6p + 2a + (side > 0)] is a leaf of the same level appears in that
// neighbour's ghost layer at box coordinate c_a - 9 (side +1) or c_a + 9 (side -1).  0: no copy.
__device__ __forceinline__ void push_offsets(const int32_t *__restrict__ nbr, int p, int x, int y, int z, int o,
                                             int64_t pd[3], int axes = 7)
{
    const int c[3] = {x, y, z};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        pd[a] = 0;
        if (!nbr || !((axes >> a) & 1)) continue;
        const int side = c[a] >= 9 ? 1 : (c[a] <= 5 ? -1 : 0);
        if (side == 0) continue;
        const int np = nbr[p * 6 + 2 * a + (side > 0 ? 1 : 0)];
        if (np < 0) continue;
        int m[3] = {x, y, z};
        m[a] = side > 0 ? c[a] - 9 : c[a] + 9;
        pd[a] = (int64_t)(np - p) * PS + (boff(m[0], m[1], m[2]) - o);
    }
}

// Whole rows.  A row's nine interior cells are 72 of its line's 128 bytes, and a line written in part
// costs memory 2.4 times a whole one (rows of 4 GiB: 1.81 against 0.75 ms; it is read back to be
// completed).  Where the output is a work buffer of a closed step, whose same-level x halos nobody reads,
// the first seven lanes of a row therefore store their value once more, over the row's other seven
// elements (x halo and padding): this returns where, relative to the lane's own cell at x.  The ghosts
// of a Sommerfeld face are evolved and stay out of it; those that a fill writes are filled afterwards.
__device__ __forceinline__ int row_rest(int x, const int32_t *__restrict__ pface, int p)
{
    const int k = x - 3, to = k < 3 ? k : k + 9;  // 0, 1, 2, 12, 13, 14, 15
    if (k >= 7 || (pface && to < 15 && pface[6 * p + (k < 3 ? 0 : 1)] >= 0)) return 0;
    return to - x;
}

// Fused stage on the Sommerfeld ghosts of boundary face fi: G_L of Qs combined at once into
// stage s (one thread per ghost cell, all slots).
__device__ __forceinline__ void stage_ghost_face(int fi, int idx, int32_t s, double dt, const double *__restrict__ Qs,
                                                 const double *__restrict__ Qn, double *__restrict__ acc,
                                                 double *__restrict__ Qx, const PatchGeom *__restrict__ geom,
                                                 const BoundaryFace *__restrict__ bf, const double *__restrict__ bg,
                                                 int32_t frozen)
{
    if (idx >= NFACE) return;
    const BoundaryFace f = bf[fi];
    int L, t1, t2;
    slab_coords(f.axis, idx, L, t1, t2);
    const int cg = ghost_c(f.side, L);
    const int og = slab_off(f.axis, cg, t1, t2);
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
    const double cadv = rr / (fabs(xn) * g.dx[f.axis]), cdmp = 1.0 / rr;
    const int64_t base = (int64_t)f.patch * PS;
    const double *B = bg + (int64_t)f.bg * NV * NFACE + idx;
    const int oa = acc_ghost(f.axis, f.side, idx);
    // the slots in batches of eight, every load of a batch issued before its arithmetic and stores
    // (this work-group holds a whole CU's LDS while it runs, so it must not wait slot by slot)
    for (int v0 = 0; v0 < NV; v0 += SB8) {
        double qL[SB8], qI[SB8], qB[SB8], q0[SB8], a0[SB8];
#pragma unroll
        for (int j = 0; j < SB8; ++j) {
            const int v = v0 + j;
            if (v >= NV) break;
            qL[j] = Qs[base + v * CS + og];
            qI[j] = Qs[base + v * CS + oi];
            qB[j] = B[v * NFACE];
            q0[j] = s < 3 ? Qn[base + v * CS + og] : 0.0;
            a0[j] = s > 0 ? acc[base + v * CS + oa] : 0.0;
        }
#pragma unroll
        for (int j = 0; j < SB8; ++j) {
            const int v = v0 + j;
            if (v >= NV) break;
            const double r = (v != SK0 && !(frozen && frozen_slot(v)))
                                 ? -cadv * (qL[j] - qI[j]) - cdmp * (qL[j] - qB[j]) : 0.0;
            const int64_t e = base + v * CS + og;
            const int64_t ea = base + v * CS + oa;
            if (s == 0) {
                acc[ea] = q0[j] + (1.0 / 6.0) * dt * r;
                Qx[e] = q0[j] + 0.5 * dt * r;
            } else if (s < 3) {
                acc[ea] = a0[j] + (1.0 / 3.0) * dt * r;
                Qx[e] = q0[j] + (s == 1 ? 0.5 : 1.0) * dt * r;
            } else {
                Qx[e] = a0[j] + (1.0 / 6.0) * dt * r;
            }
        }
    }
}


// The Sommerfeld ghost cells beside z-slab sl of patch p, handled by that slab's work-group after
// its interior: of each boundary face of the patch, the ghost cells next to the slab's three planes
// (81 for an x or y face; the whole face slab of 243 for the z face below slab 0 or above slab 2).
// Those rows were just fetched and written by the same work-group, so the ghost update finds them
// in the L2 instead of touching a line of HBM for every 3 ghost cells of an x face.  cell(fi, idx)
// is called once for every such ghost cell (face fi of the boundary-face list, index idx in its slab).
template <typename Cell>
__device__ __forceinline__ void ghost_slab_cells(int p, int sl, const int32_t *__restrict__ pface, Cell &&cell)
{
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        const int fi = pface[p * 6 + f];
        const int axis = f >> 1;
        const int n = fi < 0 ? 0 : (axis < 2 ? 81 : ((f & 1) ? (sl == 2 ? NFACE : 0) : (sl == 0 ? NFACE : 0)));
        for (int r = (int)threadIdx.x; r < n; r += (int)blockDim.x) {
            // slab_coords order: x face idx = (L - 1) + 3 y + 27 z; y face idx = x + 9 z + 81 (L - 1)
            const int idx = axis == 0 ? 81 * sl + r : (axis == 1 ? 81 * (r / 27) + 27 * sl + r % 27 : r);
            cell(fi, idx);
        }
    }
}

// Right-hand side G_L of all slots at ghost cell idx of boundary face fi (what k_rhs_sommerfeld
// computes one thread per slot), the slots in batches of eight with every load of a batch first.
__device__ __forceinline__ void rhs_ghost_cell(int fi, int idx, const double *__restrict__ Q, double *__restrict__ K,
                                               const PatchGeom *__restrict__ geom,
                                               const BoundaryFace *__restrict__ bf, const double *__restrict__ bg,
                                               int32_t frozen)
{
    if (idx >= NFACE) return;
    const BoundaryFace f = bf[fi];
    int L, t1, t2;
    slab_coords(f.axis, idx, L, t1, t2);
    const int cg = ghost_c(f.side, L);
    const int og = slab_off(f.axis, cg, t1, t2);
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
    const double *Qp = Q + (int64_t)f.patch * PS;
    double *Kp = K + (int64_t)f.patch * PS;
    const double *B = bg + (int64_t)f.bg * NV * NFACE + idx;
    for (int v0 = 0; v0 < NV; v0 += SB8) {
        double qL[SB8], qI[SB8], qB[SB8];
#pragma unroll
        for (int j = 0; j < SB8; ++j) {
            const int v = v0 + j;
            if (v >= NV) break;
            qL[j] = Qp[v * CS + og];
            qI[j] = Qp[v * CS + oi];
            qB[j] = B[v * NFACE];
        }
#pragma unroll
        for (int j = 0; j < SB8; ++j) {
            const int v = v0 + j;
            if (v >= NV) break;
            Kp[v * CS + og] = (v == SK0 || (frozen && frozen_slot(v)))
                                  ? 0.0
                                  : -(rr / (fabs(xn) * g.dx[f.axis])) * (qL[j] - qI[j]) - (1.0 / rr) * (qL[j] - qB[j]);
        }
    }
}


}  // namespace ccz4
