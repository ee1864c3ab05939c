// The LDS-staged right-hand-side and fused-stage kernels, and their launches for one algebra type and
// advection stencil.  Each (type, stencil) is a translation unit of its own (ccz4_lds_*.hip): the
// kernels are long straight-line programs, and the four compile side by side.
#pragma once
#include <hip/hip_runtime.h>

#include "ccz4_device.hpp"
#include "ccz4_kernels.hpp"
#include "ccz4_rhs_lds.hpp"

namespace ccz4 {

// LDS-staged variants: one work-group per (patch, z-slab), every lane takes part in staging;
// the 158 KiB of LDS leave one work-group per CU, so the waves may use the whole register file.
template <int XG>
__device__ __forceinline__ void lds_cell_setup(double *lds, double *ldsb, int sl, const PatchGeom &g, const RhsParams &prm,
                                               const HaloSrc &hs, LdsCell<XG> &C, uint32_t &ob, bool &act)
{
    int x, y, zl;
    act = slab_cell((int)threadIdx.x, x, y, zl);
    C.s = lds;
    C.sb = ldsb;
    lds_cell_offsets(C, x, y, zl, hs);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        C.i12[a] = 1.0 / (12.0 * g.dx[a]);
        C.koc[a] = prm.ko_eps / (64.0 * g.dx[a]);
    }
    ob = 8u * (uint32_t)boff(x, y, zl + 3 + 3 * sl);
}

template <typename T, int LOP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void k_rhs_lds(
    const double *__restrict__ Q, double *__restrict__ K, const PatchGeom *__restrict__ geom, int32_t npatch,
    RhsParams prm, const BoundaryFace *__restrict__ bf, const double *__restrict__ bg,
    const int32_t *__restrict__ pface, int32_t linear, const int32_t *__restrict__ order)
{
    __shared__ double lds[LDS_A], ldsb[LDS_B];
    const int64_t lb = linear ? (int64_t)blockIdx.x : xcd_logical_block(blockIdx.x, gridDim.x);
    if (lb / 3 >= npatch) return;  // uniform over the work-group
    const int p = __builtin_amdgcn_readfirstlane(order[lb / 3]);
    const int sl = (int)(lb % 3);
    const PatchGeom g = geom[p];
    LdsCell<0> C;
    uint32_t ob;
    bool act;
    const HaloSrc hs{};
    lds_cell_setup(lds, ldsb, sl, g, prm, hs, C, ob, act);
    LdsRhsSink snk{PatchBuf{K + (int64_t)p * PS}, ob, prm.formulation};
    rhs_slab_lds<T, LOP, 0>(Q + (int64_t)p * PS, lds, ldsb, sl, act, ob, C, prm, snk, hs);
    if (pface) {
        const int32_t frozen = prm.shift == 0;
        ghost_slab_cells(p, sl, pface, [&](int fi, int idx) { rhs_ghost_cell(fi, idx, Q, K, geom, bf, bg, frozen); });
    }
}

// Stage sink of the LDS kernel: stage s of RK4 on a round's slots together.  Every uniform choice (the
// stage, the formulation, which faces are copied) is made once per round instead of once per slot, and
// the accesses are buffer accesses.
//
// Two forms of the combine.  Two-register (CLOSED = 0), as StageSink: acc gathers Q^n and the weighted
// right-hand sides.  Closed (CLOSED = 1), for the four stages of a step launched together, where Q_s
// is the unchanged output of the stage before: with Q1 = Q^n + dt/2 k1, Q2 = Q^n + dt/2 k2,
// Q3 = Q^n + dt k3 classical RK4 is
//   Q^{n+1} = (-Q^n + Q1 + 2 Q2 + Q3) / 3 + dt/6 k4 = A + (Q3 - A) / 3 + dt/6 k4,  A = Q2 + (Q1 - Q^n) / 2,
// so that acc (= A) is written by s = 1 and read by s = 3 only: two of its three writes and two of its
// three reads go, and Q_s itself is at hand in LDS for most slots.  The differences are of nearly
// equal numbers (exact up to the roundings of Q1..Q3), so the rounding is that of the other form.
// The line between the two (STREAM): 256 MB of last-level cache, 157 leaves.  Steps with ordinary and with
// nontemporal stores: 27 leaves 0.203 and 0.213 ms, 100 leaves 0.602 and 0.613, 125 leaves 0.692 and 0.692,
// 150 leaves 0.741 and 0.730, 4096 leaves 14.82 and 14.62, three levels in mixed precision 20.97 and 20.58.
constexpr int64_t STREAM_LEAVES = (int64_t)256 * 1024 * 1024 / (PS * 8);

template <int CLOSED, int STREAM>
struct LdsStageSink {
    PatchBuf qn, acc, qx;
    uint32_t ob, oc;   // byte offsets of the cell in a slot of the state and of the accumulator
    int s;
    int so;            // second-order formulation: the auxiliaries are left alone
    double dt;
    int64_t pd[3];     // offsets (doubles) of the cell's copies in same-level neighbours' face halos
                       // of Q_next along each axis, 0 for none
    double carry[12];  // s = 3: gt_ij and At_ij of Q^{n+1}, projected in finish()

    // The copies of slots' values in the neighbours' halos.  Those into the y and z face halos (made
    // only when a step ends) are streamed past the caches: no stage reads them (the next stage
    // gathers those halos from the neighbours' interiors) and their rows are partial lines that
    // nothing else writes, so cached they only wait in L2 as dirty lines for the next launch to evict
    // (2-3 ms per step on 24^3 patches).  The x-face copies stay cached: they complete lines of the
    // neighbour's own rows in L2.
    template <int N, typename Use>
    __device__ __forceinline__ void push(const int (&slots)[N], const double (&val)[N], Use use) const
    {
        double *const cell = const_cast<double *>(qx.base) + (ob >> 3);
#pragma unroll
        for (int a = 0; a < 3; ++a)
            if (pd[a] != 0) {
                double *const to = cell + pd[a];
#pragma unroll
                for (int j = 0; j < N; ++j)
                    if (use(slots[j])) {
                        if (a == 0) to[slots[j] * CS] = val[j];
                        else __builtin_nontemporal_store(val[j], to + slots[j] * CS);
                    }
            }
    }

    // A round's outputs in two halves: every load first, so that they are in
    // flight together, then the combines and stores.  The acc stream, and
    // Q^n at s > 0, are touched once per launch, so they go through the caches as nontemporal:
    // the lines the slab staging shares between work-groups stay in L2 longer (2-3% per stage).
    // At s = 0, Q^n is Q_s and its loads hit the lines just staged, which must stay.  Q_next keeps
    // ordinary stores where neighbours push copies into its rows, which merge in L2.  Stages 0..2 of a
    // closed step push none: their stores are nontemporal too once a state no longer fits the last-level
    // cache, where the next stage would find it (STREAM_LEAVES).
    template <int N, typename Use, typename Own>
    __device__ __forceinline__ void load_some(const int (&slots)[N], double (&a)[N], double (&b)[N], Own own,
                                              Use use) const
    {
        if (CLOSED && s != 2) {
#pragma unroll
            for (int j = 0; j < N; ++j)
                if (use(slots[j])) a[j] = own(slots[j]);
        } else if (s == 0) {
#pragma unroll
            for (int j = 0; j < N; ++j)
                if (use(slots[j])) a[j] = qn.load(ob, slots[j]);
        } else if (s < 3) {
#pragma unroll
            for (int j = 0; j < N; ++j)
                if (use(slots[j])) a[j] = qn.load<BUF_NT>(ob, slots[j]);
        }
        if (CLOSED && s == 1) {
#pragma unroll
            for (int j = 0; j < N; ++j)
                if (use(slots[j])) b[j] = qn.load<BUF_NT>(ob, slots[j]);
        } else if (CLOSED ? s == 3 : s > 0) {
#pragma unroll
            for (int j = 0; j < N; ++j)
                if (use(slots[j])) b[j] = acc.load<BUF_NT>(oc, slots[j]);
        }
    }
    template <int N, typename Use>
    __device__ __forceinline__ void store_some(const int (&slots)[N], double (&r)[N], const double (&a)[N],
                                               const double (&b)[N], Use use)
    {
        if (s < 3) {
            const double c = (s == 2 ? 1.0 : 0.5) * dt;
            if (!CLOSED) {
                const double w = (s == 0 ? 1.0 / 6.0 : 1.0 / 3.0) * dt;
                if (s == 0) {
#pragma unroll
                    for (int j = 0; j < N; ++j)
                        if (use(slots[j])) acc.store<BUF_NT>(a[j] + w * r[j], oc, slots[j]);
                } else {
#pragma unroll
                    for (int j = 0; j < N; ++j)
                        if (use(slots[j])) acc.store<BUF_NT>(b[j] + w * r[j], oc, slots[j]);
                }
            }
            if (CLOSED && s == 1) {
#pragma unroll
                for (int j = 0; j < N; ++j)
                    if (use(slots[j])) {
                        r[j] = b[j] + c * r[j];
                        acc.store<BUF_NT>(r[j] + 0.5 * (a[j] - b[j]), oc, slots[j]);
                    }
            } else {
#pragma unroll
                for (int j = 0; j < N; ++j)
                    if (use(slots[j])) r[j] = a[j] + c * r[j];
            }
#pragma unroll
            for (int j = 0; j < N; ++j)
                if (use(slots[j])) qx.store<STREAM ? BUF_NT : BUF_DEFAULT>(r[j], ob, slots[j]);
            push(slots, r, use);
        } else {
            const double w = (1.0 / 6.0) * dt;
            if (CLOSED) {
#pragma unroll
                for (int j = 0; j < N; ++j)
                    if (use(slots[j])) r[j] = (b[j] + (1.0 / 3.0) * (a[j] - b[j])) + w * r[j];
            } else {
#pragma unroll
                for (int j = 0; j < N; ++j)
                    if (use(slots[j])) r[j] = b[j] + w * r[j];
            }
#pragma unroll
            for (int j = 0; j < N; ++j)
                if (use(slots[j])) {
                    const int v = slots[j];
                    if (projected(v)) carry[v < 6 ? v : v - SAT + 6] = r[j];
                    else qx.store(r[j], ob, v);
                }
            push(slots, r, [&](int v) { return use(v) && !projected(v); });
        }
    }
    static __device__ __forceinline__ constexpr bool projected(int v) { return v < 6 || (v >= SAT && v < SAT + 6); }
    template <int N, typename Own>
    __device__ __forceinline__ void load(const int (&slots)[N], double (&a)[N], double (&b)[N], Own own) const
    {
        load_some(slots, a, b, own, [](int v) { return !aux_slot(v); });
        if (!so) load_some(slots, a, b, own, [](int v) { return aux_slot(v); });
    }
    template <int N>
    __device__ __forceinline__ void store(const int (&slots)[N], double (&r)[N], const double (&a)[N],
                                          const double (&b)[N])
    {
        store_some(slots, r, a, b, [](int v) { return !aux_slot(v); });
        if (!so) store_some(slots, r, a, b, [](int v) { return aux_slot(v); });
    }
    __device__ __forceinline__ void finish()
    {
        if (s != 3) return;
        constexpr int slots[12] = {SG, SG + 1, SG + 2, SG + 3, SG + 4, SG + 5, SAT, SAT + 1, SAT + 2, SAT + 3, SAT + 4, SAT + 5};
        double q[SAT + 6], out[12];
#pragma unroll
        for (int j = 0; j < 12; ++j) q[slots[j]] = carry[j];
        project_cell(q);
#pragma unroll
        for (int j = 0; j < 12; ++j) {
            out[j] = q[slots[j]];
            qx.store(out[j], ob, slots[j]);
        }
        push(slots, out, [](int) { return true; });
    }
};

template <typename T, int LOP, int CLOSED, int STREAM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void k_stage_lds(
    const double *__restrict__ Qs, const double *__restrict__ Qn, double *__restrict__ acc, double *__restrict__ Qx,
    const PatchGeom *__restrict__ geom, int32_t npatch, int32_t nb_slab, RhsParams prm, int32_t s, double dt,
    const BoundaryFace *__restrict__ bf, const double *__restrict__ bg, const int32_t *__restrict__ pface,
    const int32_t *__restrict__ nbr, int32_t paxes, int32_t gaxes, int32_t linear,
    const int32_t *__restrict__ order)
{
    __shared__ double lds[LDS_A], ldsb[LDS_B];
    const int64_t lb = linear ? (int64_t)blockIdx.x : xcd_logical_block(blockIdx.x, nb_slab);
    if (lb / 3 >= npatch) return;  // uniform over the work-group
    const int p = __builtin_amdgcn_readfirstlane(order[lb / 3]);
    const int sl = (int)(lb % 3);
    const PatchGeom g = geom[p];
    LdsCell<CLOSED> C;
    uint32_t ob;
    bool act;
    const HaloSrc hs = halo_sources(nbr, p, gaxes);
    lds_cell_setup(lds, ldsb, sl, g, prm, hs, C, ob, act);
    LdsStageSink<CLOSED, STREAM> snk;
    snk.qn.base = Qn + (int64_t)p * PS;
    snk.acc.base = acc + (int64_t)p * PS;
    snk.qx.base = Qx + (int64_t)p * PS;
    snk.ob = ob;
    snk.oc = 8u * (uint32_t)acc_cell(sl, act ? (int)threadIdx.x : 242);
    snk.s = s;
    snk.so = prm.formulation;
    snk.dt = dt;
    {
        int x, y, zl;
        (void)slab_cell((int)threadIdx.x, x, y, zl);
        push_offsets(paxes ? nbr : nullptr, p, x, y, zl + 3 + 3 * sl, (int)(ob >> 3), snk.pd, paxes);
    }
    rhs_slab_lds<T, LOP, CLOSED>(Qs + (int64_t)p * PS, lds, ldsb, sl, act, ob, C, prm, snk, hs);
    if (pface) {
        const int32_t frozen = prm.shift == 0;
        ghost_slab_cells(p, sl, pface, [&](int fi, int idx) {
            stage_ghost_face(fi, idx, s, dt, Qs, Qn, acc, Qx, geom, bf, bg, frozen);
        });
    }
}

template <typename T, int LOP>
hipError_t launch_rhs_lds(const RhsLaunch &a, hipStream_t st)
{
    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_rhs_lds<T, LOP>), dim3((unsigned)a.blocks), dim3(256), 0, st, a.Q, a.K, a.geom,
                       a.npatch, a.p, a.bf, a.bg, a.pface, a.linear, a.order);
    return hipGetLastError();
}

template <typename T, int LOP>
hipError_t launch_stage_lds(const StageLaunch &a, hipStream_t st)
{
    const dim3 g((unsigned)a.blocks), b(256);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, g, b, 0, st, a.Qs, a.Qn, a.acc, a.Qx, a.geom, a.npatch, a.blocks, a.p, a.s, a.dt, a.bf,
                           a.bg, a.pface, a.nbr, a.paxes, a.gaxes, a.linear, a.order);
    };
    if (!a.closed) go(k_stage_lds<T, LOP, 0, 0>);
    else if (a.s < 3 && a.npatch > STREAM_LEAVES) go(k_stage_lds<T, LOP, 1, 1>);
    else go(k_stage_lds<T, LOP, 1, 0>);
    return hipGetLastError();
}

}  // namespace ccz4
