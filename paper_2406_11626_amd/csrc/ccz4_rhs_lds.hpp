// LDS-staged evaluation of the first-order CCZ4 right-hand side for one z-slab of a patch
// (3 x 9 x 9 = 243 cells, one work-group of 256 threads).
//
// Every evolved slot is copied once per evaluation from the patch box into LDS with gfx950's
// direct global->LDS loads (16 bytes per lane, no registers involved), in parts of at most nine
// slots.  A slot occupies, in LDS, the slab's three planes in box layout (3 x 15 x 18 doubles,
// carrying the x and y halos) followed by the interior rows of the three planes below and the
// three planes above the slab (6 x 9 rows x 10 doubles, columns x = 2..11).  Each face
// halo is read either from the patch's own halo or straight from the interior of the same-level
// neighbour across that face (HaloSrc).  Every FD4
// derivative and Kreiss-Oliger sum is then read from LDS; a per-lane table maps the seven
// z-neighbours of a cell into the own planes or the halo rows.
//
// There is room for fifteen slots and for one work-group per CU, one wave per SIMD, so nothing but the
// work-group's own next copies can fill the time it computes.  The buffers therefore form two groups, of
// nine and six slots, that take turns: while the lanes work on one group, the next part of the slots is
// copied into the other (all fifteen buffers filled, waited for and used in turn before: right-hand side
// of 1287 leaves 1.02 -> 0.98 ms, step on 4096 leaves 15.77 -> 15.27 ms, in mixed precision 15.25 ->
// 14.75 ms, of the second-order formulation 17.2 -> 16.6 ms).
//
// The order of the equations is chosen so that each slot is staged exactly once:
//   round 1: B | At     -> d tr(At), the shift-derivative contractions, the non-advective part of
//                          the D equations, advection + KO of At and B (kept in registers)
//   round 2: D (9 | 6)  -> contractions G1, H, U, E of d D; outputs of those D slots
//   round 3: D (3), P, A | Ghat, K, Theta
//                       -> last contractions and D outputs; Ricci tensor, nabla nabla alpha and
//                          the Z terms; outputs At, K, Theta, Ghat, A, P; B and b without d b
//   round 4: b, gt | alpha, beta, phi
//                       -> outputs B, b, gt, alpha, beta, phi and K_0 = 0
// The algebra is the one of ccz4_rhs_phased.hpp, term for term (App. B); T is double, or float
// for the mixed-precision mode with the same split between FP64 and FP32 parts.
#pragma once
#include <type_traits>

#include "ccz4_rhs_phased.hpp"

namespace ccz4 {

// A staged row of the own planes is 18 doubles, in one of two layouts (XG, a template parameter):
//   XG = 0: the patch's own row, x = 0..15 (the ninth pair repeats the eighth): every neighbour of a
//           cell along x at a fixed distance.
//   XG = 1: the x halos may be gathered from the neighbours.  Columns 0..3: the x- halo group, 4..13:
//           x = 2..11 of the patch, 14..17: the x+ halo group.  A halo group is two 16-byte pairs: the
//           patch's own (x = 0..3; x = 12..15), or the pairs of the neighbour's interior that hold the
//           three cells (x = 8..11 of the x- neighbour; x = 2..5 of the x+ one).  Interior cells sit at
//           x + 2; a halo cell of the x- face at x (own) or x + 1 (gathered), of the x+ face at x + 2
//           or x + 3: a per-lane table (LdsCell::xo), whose six base registers cost the merged reads of
//           XG = 0 (right-hand side alone: 2.98 against 3.07 ms on 4096 leaves), which the copies that
//           a step then does not make pay for (a step: 18.1 -> 16.2 ms).
// The pitch of 18 doubles (an odd number of pairs) spreads the rows of a wave's reads over the banks.
constexpr int LROW = 18;
constexpr int LPAIRS = LROW / 2;                  // 16-byte copies per staged row
constexpr int LPLANE = NBX * LROW;                // one staged plane, 15 rows
constexpr int LDS_OWN = 3 * LPLANE;               // the slab's planes
constexpr int LDS_OWN_PAIRS = 3 * NBX * LPAIRS;   // 405 copies
constexpr int LDS_HROW = 10;                      // halo row: x = 2..11 (16-byte aligned pairs)
constexpr int LDS_HALO = 6 * 9 * LDS_HROW;        // 540 doubles
constexpr int LDS_SLOT = LDS_OWN + LDS_HALO;      // 1350 doubles
constexpr int LDS_NBUF = 15;
// The buffers lie in two LDS variables, 0..8 and 9..14: a wait for the copies into one then leaves those
// into the other in flight (the compiler tracks them by variable).
constexpr int LDS_NA = 9, LDS_NB = LDS_NBUF - LDS_NA;
constexpr int LDS_A = LDS_NA * LDS_SLOT, LDS_B = LDS_NB * LDS_SLOT;  // 97200 and 64800 bytes

typedef __attribute__((address_space(3))) void lds_void_t;

// One patch of a state (or of the accumulator), addressed as a buffer: a uniform base, a byte offset
// per lane within a slot (8 o, the same for every slot) and the slot's byte offset in a scalar
// register, so that no access needs vector address arithmetic (64-bit adds on a slot stride beyond
// the instructions' immediate range took two vector instructions per access and array).
typedef unsigned int buf_b64_t __attribute__((ext_vector_type(2)));
constexpr int BUF_DEFAULT = 0, BUF_NT = 2;  // cache policy: default, nontemporal

struct PatchBuf {
    const double *base;
    template <int POLICY = BUF_DEFAULT>
    __device__ __forceinline__ double load(uint32_t ob, int v) const
    {
        return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rsrc(), ob, v * CS * 8, POLICY));
    }
    template <int POLICY = BUF_DEFAULT>
    __device__ __forceinline__ void store(double x, uint32_t ob, int v) const
    {
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(buf_b64_t, x), rsrc(), ob, v * CS * 8, POLICY);
    }
    __device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc() const
    {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<double *>(base), 0, (int)(PS * 8), 0x00027000);
    }
};

// Where the face halos of a patch are read from: d[2 a + (side > 0)] is added to the element index of
// a halo cell of the face of axis a on that side.  0 reads the patch's own halo (filled beforehand);
// for a same-level neighbour n the offset reads the neighbour's interior cell at the same position,
// so that those halos need no copy: (n - p) PS -+ 9 stride_a for y and z.  An x group is whole 16-byte
// pairs, which in the neighbour begin one cell lower: (n - p) PS + 8 (x-) and (n - p) PS - 10 (x+).
struct HaloSrc {
    int64_t d[6];
};

// The sources of patch p's halos with the faces of the axes in gaxes gathered from same-level
// neighbours (nbr: the leaves' face neighbours, -1 where there is none of the same level).
__device__ __forceinline__ HaloSrc halo_sources(const int32_t *__restrict__ nbr, int p, int32_t gaxes)
{
    HaloSrc hs;
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        const int a = f >> 1;
        const int n = (gaxes >> a) & 1 ? __builtin_amdgcn_readfirstlane(nbr[p * 6 + f]) : -1;
        const int64_t step = a == 0 ? ((f & 1) ? -10 : 8) : ((f & 1) ? -9 : 9) * (a == 1 ? YS : ZS);
        hs.d[f] = n >= 0 ? (int64_t)(n - p) * PS + step : 0;
    }
    return hs;
}

// The staging copies of one lane.  A slot's LDS_PAIRS 16-byte pairs (own planes first: 45 rows of
// LPAIRS pairs; then the
// halo rows: pair e being plane e / 45 (0..2 below, 3..5 above), row (e / 5) % 9, columns
// 2 + 2 (e % 5)) are contiguous in LDS, so wave w copies chunks w, w + 4, w + 8 of 64 pairs.  The
// source addresses of a lane's copies are the same in every slot up to the slot stride: they are
// formed once per work-group instead of once per copy (which took about 25 integer instructions a
// copy, 4000 of the 10,900 vector instructions of a right-hand side per wave).
constexpr int LDS_PAIRS = LDS_SLOT / 2;
constexpr int LDS_COPIES = (LDS_PAIRS + 255) / 256;  // per lane; the last only where pair < LDS_PAIRS
static_assert(LDS_COPIES == 3, "three copies per lane and slot");

struct Stager {
    const double *src[LDS_COPIES];  // the lane's sources in slot 0
    bool last;                      // the lane takes part in its wave's last chunk
    int wave;                       // uniform
};

// slab sl of the patch at qp; the rows y <= 2 and y >= 12 come from the y faces' sources, planes
// outside the patch from the z faces' sources (the x halos of those rows are never read: with XG
// their pairs repeat the row's first and last interior ones)
template <int XG>
__device__ __forceinline__ Stager lds_stager(const double *__restrict__ qp, int sl, const HaloSrc &hs)
{
    Stager g;
    g.wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
#pragma unroll
    for (int i = 0; i < LDS_COPIES; ++i) {
        const int q = min(i * 256 + (int)threadIdx.x, LDS_PAIRS - 1);
        int e;
        int64_t d;  // selects, not an index into hs.d: a lane-dependent index would put the array in memory
        if (q < LDS_OWN_PAIRS) {
            const int r = q / LPAIRS, j = q % LPAIRS, y = r % 15;
            int x;
            if (XG) {
                const bool in = y >= 3 && y <= 11, lo = j < 2, hi = j >= 7;
                d = y <= 2 ? hs.d[2] : (y >= 12 ? hs.d[3] : (lo ? hs.d[0] : (hi ? hs.d[1] : 0)));
                x = lo ? (in ? 2 * j : 2) : (hi ? (in ? 2 * j - 2 : 10) : 2 * j - 2);
            } else {
                d = y <= 2 ? hs.d[2] : (y >= 12 ? hs.d[3] : 0);
                x = 2 * (j < 8 ? j : 7);
            }
            e = (3 + 3 * sl) * ZS + r * XS + x;
        } else {
            const int h = q - LDS_OWN_PAIRS, hp = h / 45, row = (h / 5) % 9, pr = h % 5;
            const int z = hp < 3 ? 3 * sl + hp : 3 * sl + 3 + hp;
            e = z * ZS + (row + 3) * YS + 2 + 2 * pr;
            d = z <= 2 ? hs.d[4] : (z >= 12 ? hs.d[5] : 0);
        }
        g.src[i] = qp + e + d;
    }
    g.last = (LDS_COPIES - 1) * 256 + (int)threadIdx.x < LDS_PAIRS;
    return g;
}

// Ends a group of copies: those issued after it stay after it, which the counts of wait_memory rest on (the
// groups write different LDS variables, so nothing else keeps the compiler from mixing them).
__device__ __forceinline__ void copies_issued() { asm volatile("" ::: "memory"); }

// Issue the direct global->LDS copies of N slots into the buffers at `lds`, which no wave reads any
// more (lds_swap); returns without waiting for them.
template <int N>
__device__ __forceinline__ void lds_issue(double *lds, const int (&slots)[N], const Stager &g)
{
    double *dst = lds + g.wave * 128;
#pragma unroll
    for (int j = 0; j < N; ++j)
#pragma unroll
        for (int i = 0; i < LDS_COPIES - 1; ++i)
            __builtin_amdgcn_global_load_lds((const void *)(g.src[i] + slots[j] * CS),
                                             (lds_void_t *)(dst + j * LDS_SLOT + i * 512), 16, 0, 0);
    if (g.last)
#pragma unroll
        for (int j = 0; j < N; ++j)
            __builtin_amdgcn_global_load_lds((const void *)(g.src[LDS_COPIES - 1] + slots[j] * CS),
                                             (lds_void_t *)(dst + j * LDS_SLOT + (LDS_COPIES - 1) * 512), 16, 0, 0);
    copies_issued();
}

// Wait until at most N (0..63) memory operations of the wave are outstanding: all but its last N, in the
// order of their issue, have landed.
template <int N>
__device__ __forceinline__ void wait_memory()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((N & 15) | (N >> 4) << 14 | 0x0f70);
    asm volatile("" ::: "memory");
}

// Wait for every copy but those of the last group, of these slots (a wave without a share in the last chunk
// issues LDS_COPIES - 1 a slot, the others more).
template <int N>
__device__ __forceinline__ void wait_all_but(const int (&)[N])
{
    wait_memory<(LDS_COPIES - 1) * N>();
}

// Work-group barrier that orders LDS reads and copies only: each wave's LDS reads are done, and the
// copies that it waited for have landed for all (__syncthreads would wait for everything in flight).
__device__ __forceinline__ void lds_swap()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);  // LDS reads
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// One cell's view of the staged slab.
template <int XG>
struct LdsCell {
    const double *s, *sb;  // LDS buffers 0..8, and the others
    int c;            // index of the cell in the own planes: zl * LPLANE + y * LROW + x (+ 2 with XG)
    int xo[7];        // with XG, index of the x-neighbour at offset k - 3
    int zo[7];        // index of the z-neighbour at offset k - 3
    double i12[3];    // 1 / (12 dx_a)
    double koc[3];    // eps / (64 dx_a)
};

template <int XG>
__device__ __forceinline__ double lv(const LdsCell<XG> &c, int b, int a, int k)
{
    const double *f = b < LDS_NA ? c.s + b * LDS_SLOT : c.sb + (b - LDS_NA) * LDS_SLOT;
    return k == 0 ? f[c.c]
                  : (a == 0 ? f[XG ? c.xo[k + 3] : c.c + k] : (a == 1 ? f[c.c + k * LROW] : f[c.zo[k + 3]]));
}

// Box coordinates x, y and plane zl of the cell that lane tid (0..255) of a slab's work-group takes
// (the order of slab_row_y; idle lanes repeat the last cell).
__device__ __forceinline__ bool slab_cell(int tid, int &x, int &y, int &zl)
{
    const bool act = tid < 243;
    const int cc = act ? tid : 242, m = cc / 9;
    zl = m / 9;
    x = cc % 9 + 3;
    y = slab_row_y(zl, m % 9) + 3;
    return act;
}

// The LDS offsets of cell (x, y) (box indices) in plane zl (0..2) of the staged slab: its own
// index, those of its x-neighbours (own columns, or the halo groups; hs tells which are gathered) and
// those of its z-neighbours (own planes, or the halo rows below and above).
template <int XG>
__device__ __forceinline__ void lds_cell_offsets(LdsCell<XG> &C, int x, int y, int zl, const HaloSrc &hs)
{
    const int row = zl * LPLANE + y * LROW, own = XG ? 2 : 0;
    const int lo = XG && hs.d[0] != 0 ? 1 : 0, hi = XG ? (hs.d[1] != 0 ? 3 : 2) : 0;
    C.c = row + x + own;
#pragma unroll
    for (int k = -3; k <= 3; ++k) {
        const int x2 = x + k, z2 = zl + k;
        C.xo[k + 3] = row + x2 + (x2 < 3 ? lo : (x2 > 11 ? hi : own));
        C.zo[k + 3] = (z2 >= 0 && z2 <= 2) ? z2 * LPLANE + y * LROW + x + own
                                            : LDS_OWN + (z2 < 0 ? z2 + 3 : z2) * 90 + (y - 3) * LDS_HROW + (x - 2);
    }
}

// The 19 points that the differences of one staged slot take, read from LDS at once (the compiler barrier
// keeps the reads of one slot from being hoisted above those of the one before).
struct Points {
    double q[3][6], own;
    double i12[3], koc[3];  // of the cell
};

template <int XG>
__device__ __forceinline__ Points points(const LdsCell<XG> &c, int b)
{
    Points r;
    r.own = lv(c, b, 0, 0);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
#pragma unroll
        for (int k = 0; k < 6; ++k) r.q[a][k] = lv(c, b, a, k < 3 ? k - 3 : k - 2);
        r.i12[a] = c.i12[a];
        r.koc[a] = c.koc[a];
    }
    asm volatile("" ::: "memory");
    return r;
}
__device__ __forceinline__ double lv(const Points &p, int, int a, int k)
{
    return k == 0 ? p.own : p.q[a][k < 0 ? k + 3 : k + 2];
}

// Calls f(n, points of buffer b + n) for n = 0..N - 1, a slot's points read while the one before it is
// worked on, one read to three vector instructions: the work-group's four waves leave every barrier
// together and would otherwise take turns, all queueing at the LDS and then all computing (right-hand
// side of 1287 leaves 0.98 -> 0.96 ms; a fused stage, bound by memory, gains nothing).
template <int N, int XG, typename F>
__device__ __forceinline__ void each_slot(const LdsCell<XG> &C, int b, F f)
{
    Points cur = points(C, b);
#pragma unroll
    for (int n = 0; n < N; ++n) {
        Points next = cur;
        if (n + 1 < N) next = points(C, b + n + 1);
        f(n, cur);
#pragma unroll
        for (int k = 0; k < 17; ++k) {  // one LDS read, three vector instructions
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        cur = next;
    }
}

template <typename Cell>
__device__ __forceinline__ double fd(const Cell &c, int b, int a)
{
    return (8.0 * (lv(c, b, a, 1) - lv(c, b, a, -1)) - (lv(c, b, a, 2) - lv(c, b, a, -2))) * c.i12[a];
}

template <typename Cell>
__device__ __forceinline__ double ko_axis_lds(const Cell &c, int b, int a)
{
#if CCZ4_KO_PRINTED_ORDER
#pragma clang fp contract(off)
    return lv(c, b, a, -3) - 6.0 * lv(c, b, a, -2) + 15.0 * lv(c, b, a, -1) - 20.0 * lv(c, b, a, 0) +
           15.0 * lv(c, b, a, 1) - 6.0 * lv(c, b, a, 2) + lv(c, b, a, 3);
#else
    const double p3 = lv(c, b, a, -3) + lv(c, b, a, 3), p2 = lv(c, b, a, -2) + lv(c, b, a, 2),
                 p1 = lv(c, b, a, -1) + lv(c, b, a, 1);
    return fma(-20.0, lv(c, b, a, 0), fma(15.0, p1, fma(-6.0, p2, p3)));
#endif
}

template <typename Cell>
__device__ __forceinline__ double ko(const Cell &c, int b)
{
    const double kx = c.koc[0] * ko_axis_lds(c, b, 0), ky = c.koc[1] * ko_axis_lds(c, b, 1),
                 kz = c.koc[2] * ko_axis_lds(c, b, 2);
    return (kx + ky) + kz;
}

// Output sinks of the slab evaluation receive the complete right-hand sides (algebra, advection and
// KO) of the lane's cell, a round's slots at a time.
struct LdsRhsSink {
    PatchBuf kb;
    uint32_t ob;
    int so;  // second-order formulation: the auxiliaries' right-hand sides are 0
    __device__ __forceinline__ void finish() {}
    // A round's outputs in two halves (see rhs_slab_lds): the RHS alone reads nothing.
    template <int N, typename Own>
    __device__ __forceinline__ void load(const int (&)[N], double (&)[N], double (&)[N], Own) {}
    // K is written once and not read again in this launch, and no other work-group writes the
    // same lines: nontemporal stores keep the staged lines in L2 (2% per launch).
    template <int N>
    __device__ __forceinline__ void store(const int (&slots)[N], double (&r)[N], const double (&)[N],
                                          const double (&)[N])
    {
        if (so)
#pragma unroll
            for (int j = 0; j < N; ++j)
                if (aux_slot(slots[j])) r[j] = 0.0;
#pragma unroll
        for (int j = 0; j < N; ++j) kb.store<BUF_NT>(r[j], ob, slots[j]);
    }
};

// (s, d) of the symmetric index s = sym(cc, dd), cc <= dd
__device__ __forceinline__ constexpr int sym_first(int s) { return s < 3 ? 0 : (s < 5 ? 1 : 2); }
__device__ __forceinline__ constexpr int sym_second(int s) { return s < 3 ? s : (s < 5 ? s - 2 : 2); }

template <typename T>
__device__ __forceinline__ void dD_accumulate(const double d[3], int j, const T ig[6], T G1[3][3], T H[3][3],
                                              T U[3][3], T E[6])
{
    const int b = j / 6, s = j % 6;  // D_b,s with s = sym(cc, dd)
    const int cc = sym_first(s), dd = sym_second(s);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const T v = cvt<T>(d[a]);
        G1[b][cc] += ig[sym(a, dd)] * v;
        H[a][cc] += ig[sym(b, dd)] * v;
        if (cc != dd) {
            G1[b][dd] += ig[sym(a, cc)] * v;
            H[a][dd] += ig[sym(b, cc)] * v;
            U[a][b] += T(2) * ig[s] * v;
        } else {
            U[a][b] += ig[s] * v;
        }
        E[s] += ig[sym(a, b)] * v;
    }
}

// An opaque copy of the cell's offsets, so that loads of one block of the algebra are neither
// merged with nor hoisted above those of another (this bounds the registers each block holds).
template <int XG>
__device__ __forceinline__ LdsCell<XG> fresh(const LdsCell<XG> &c)
{
    LdsCell<XG> r = c;
    asm volatile("" : "+v"(r.c));
#pragma unroll
    for (int k = 0; k < 7; ++k) {
        if (k == 3) continue;
        if (XG) asm volatile("" : "+v"(r.xo[k]));
        asm volatile("" : "+v"(r.zo[k]));
    }
    return r;
}

__device__ __forceinline__ uint32_t fresh(uint32_t ob)
{
    asm volatile("" : "+v"(ob));
    return ob;
}

__device__ __forceinline__ double fresh(double x)
{
    asm volatile("" : "+v"(x));
    return x;
}

__device__ __forceinline__ float fresh(float x)
{
    asm volatile("" : "+v"(x));
    return x;
}

// The pointwise metric of the cell, its slots read by ld(v): g, its inverse and its determinant.
template <typename T, typename Ld>
__device__ __forceinline__ void load_metric_with(Ld ld, double gd[6], double igd[6], double &detg, T g[6], T ig[6])
{
#pragma unroll
    for (int s = 0; s < 6; ++s) gd[s] = ld(SG + s);
    metric_inverse(gd, igd, detg);
#pragma unroll
    for (int s = 0; s < 6; ++s) {
        g[s] = cvt<T>(gd[s]);
        ig[s] = cvt<T>(igd[s]);
    }
}

// The LDS buffer that holds slot v during round r of rhs_slab_lds, or -1 (see the round lists).
__device__ __forceinline__ constexpr int round_buffer(int r, int v)
{
    if (r == 1) return (v >= SAT && v < SAT + 6) ? LDS_NA + v - SAT : -1;  // At's part: B's buffers are reused
    if (r == 2) return v >= SD && v < SD + 15 ? v - SD : -1;
    if (r == 3)
        return (v >= SD + 15 && v < SD + 18) ? v - SD - 15
               : (v >= SP && v < SP + 3)     ? 3 + v - SP
               : (v >= SA && v < SA + 3)     ? 6 + v - SA
               : (v >= SGHAT && v < SGHAT + 3) ? 9 + v - SGHAT
               : v == SK                     ? 12
               : v == STHETA                 ? 13
                                             : -1;
    if (r == 4)
        return (v >= SBB && v < SBB + 3)     ? v - SBB
               : (v >= SG && v < SG + 6)     ? 3 + v - SG
               : v == SALPHA                 ? 9
               : (v >= SBETA && v < SBETA + 3) ? 10 + v - SBETA
               : v == SPHI                   ? 13
                                             : -1;
    return -1;
}

// Pointwise value of slot v at the lane's cell during round R: from the staged copy in LDS when
// the round stages v (the same double), else from the patch.
template <int R, int XG>
__device__ __forceinline__ double pw(const PatchBuf &qp, uint32_t ob, const LdsCell<XG> &C, int v)
{
    const int b = round_buffer(R, v);
    if (b >= 0) return lv(C, b, 0, 0);
    return qp.load(ob, v);
}

// The three FD4 derivatives and the Kreiss-Oliger sum of staged buffer b at the lane's cell,
// from the 19 distinct stencil points; the compiler barrier after the reads keeps the LDS
// loads of one slot from being hoisted above those of the previous one.
struct SlotDeriv {
    double d[3];
    double k;
    double a;  // advection beta^k d_k (central or lopsided), with the 4-argument form only
};

template <typename Cell>
__device__ __forceinline__ SlotDeriv stencils(const Cell &c, int b = 0)
{
    SlotDeriv r;
#pragma unroll
    for (int a = 0; a < 3; ++a) r.d[a] = fd(c, b, a);
    r.k = ko(c, b);
    r.a = 0.0;
    CCZ4_PHASE_BARRIER();
    return r;
}

// ... and the advection term with shift be: the central derivatives (LOP = 0), or the lopsided
// stencils of App. D (LOP = 1, pairing `mode` as RhsParams::advection) from the same staged
// points.  LOP is a template parameter so that the central kernel carries no lopsided code.
template <int LOP, typename Cell>
__device__ __forceinline__ SlotDeriv stencils(const Cell &c, int b, const double be[3], int32_t mode)
{
    SlotDeriv r;
#pragma unroll
    for (int a = 0; a < 3; ++a) r.d[a] = fd(c, b, a);
    r.k = ko(c, b);
    if constexpr (!LOP) {
        r.a = be[0] * r.d[0] + be[1] * r.d[1] + be[2] * r.d[2];
    } else {
        double s[3];
#pragma unroll
        for (int a = 0; a < 3; ++a)
            s[a] = lop_from_central(r.d[a], lop_use_right(mode, be[a]), lv(c, b, a, -3), lv(c, b, a, -2),
                                    lv(c, b, a, -1), lv(c, b, a, 0), lv(c, b, a, 1), lv(c, b, a, 2), lv(c, b, a, 3),
                                    c.i12[a]);
        r.a = be[0] * s[0] + be[1] * s[1] + be[2] * s[2];
    }
    CCZ4_PHASE_BARRIER();
    return r;
}

// r = v, materialised here: the opaque move keeps the computation of v inside its block of
// the algebra instead of letting it drift towards the round's output loop.
__device__ __forceinline__ void keep(double &r, double v)
{
    r = v;
    asm volatile("" : "+v"(r));
}

// Round 3's Ghat^i sector: its right-hand side (ro3[11..13]), the part of b^i's right-hand side it
// shares (rGb) and the pointwise part of the gt_ij equation (pwG), from the cell's metric, D, At,
// B, A, P / phi, the Christoffel symbols and Z, and the contractions carried from rounds 1 and 2.
template <typename T, int LOP, int XG>
__device__ __forceinline__ void ghat_sector(const LdsCell<XG> &C, const RhsParams &p, const double be[3], const T g[6],
                                            const T ig[6], const double gd[6], double detg, const T (&D)[3][6],
                                            const T (&Gt)[3][6], const T Gtv[3], const T At[6], const T (&Am)[3][3],
                                            const T (&Bm)[3][3], const T A[3], const T Ph[3], T trB, T al, T Kt, T Th,
                                            const T Zl[3], const T GB[3], const T sdBtr[3], const T dtrA[3], T red,
                                            T sfac, double (&ro3)[20], double (&rGb)[3], double (&pwG)[6])
{
    T Aup[6];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = i; j < 3; ++j)
            Aup[sym(i, j)] = Am[i][0] * ig[sym(0, j)] + Am[i][1] * ig[sym(1, j)] + Am[i][2] * ig[sym(2, j)];
    const T kap1 = cvt<T>(p.kappa1), kap3 = cvt<T>(p.kappa3);
    T dTh[3], dK[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        dTh[k] = cvt<T>(fd(C, 13, k));
        dK[k] = cvt<T>(fd(C, 12, k));
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        T t = GB[i];
        T u = T(0);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const T igik = ig[sym(i, k)];
            t += T(2) * al * igik * (dTh[k] + red * dtrA[k]) - T(4.0 / 3.0) * al * igik * dK[k];
            t += sfac * T(1.0 / 3.0) * igik * sdBtr[k];
            t += T(-2) * igik * (Th * A[k] + T(2.0 / 3.0) * al * Kt * Zl[k] + al * kap1 * Zl[k]);
            u += igik * Zl[k];
        }
        t += T(2.0 / 3.0) * Gtv[i] * trB - (Gtv[0] * Bm[0][i] + Gtv[1] * Bm[1][i] + Gtv[2] * Bm[2][i]);
        T ga = tr6(Aup, Gt[i]) - T(3) * (Aup[sym(i, 0)] * Ph[0] + Aup[sym(i, 1)] * Ph[1] + Aup[sym(i, 2)] * Ph[2]);
        t += T(2) * al * ga;
        t += T(-2) * (Aup[sym(i, 0)] * A[0] + Aup[sym(i, 1)] * A[1] + Aup[sym(i, 2)] * A[2]);
        T zb = T(0);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const T zk = ig[sym(k, 0)] * Zl[0] + ig[sym(k, 1)] * Zl[1] + ig[sym(k, 2)] * Zl[2];
            zb += zk * Bm[k][i];
        }
        t += T(2) * kap3 * (T(2.0 / 3.0) * u * trB - zb);
        const SlotDeriv sG = stencils<LOP>(C, 9 + i, be, p.advection);
        const double advG = sG.a;
        const double rG = advG + static_cast<double>(t);
        keep(ro3[11 + i], rG + sG.k);
        rGb[i] = rG - advG;
    }
    // gt_ij: 2 beta^k D_kij + gt_ki B_j^k + gt_kj B_i^k - 2/3 gt_ij tr B - 2 alpha (At_ij - gt_ij tr At / 3)
    // - (det gt - 1) gt_ij / tau
    T bet[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) bet[k] = cvt<T>(be[k]);
    const T trAt = tr6(ig, At);
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = i; j < 3; ++j) {
            const int ij = sym(i, j);
            T t = T(2) * (bet[0] * D[0][ij] + bet[1] * D[1][ij] + bet[2] * D[2][ij]);
#pragma unroll
            for (int k = 0; k < 3; ++k) t += g[sym(k, i)] * Bm[j][k] + g[sym(k, j)] * Bm[i][k];
            t += T(-2.0 / 3.0) * g[ij] * trB;
            t += T(-2) * al * (At[ij] - T(1.0 / 3.0) * g[ij] * trAt);
            keep(pwG[ij], static_cast<double>(t) - (detg - 1.0) / p.tau * gd[ij]);
        }
}

// Output slots of rounds 2, 3 and 4, in the order of the round's output buffer.
__device__ constexpr int R3_OUT[20] = {SD + 15, SD + 16, SD + 17, SAT, SAT + 1, SAT + 2, SAT + 3,
                                       SAT + 4, SAT + 5, SK, STHETA, SGHAT, SGHAT + 1, SGHAT + 2,
                                       SA, SA + 1, SA + 2, SP, SP + 1, SP + 2};
__device__ constexpr int R4_OUT[24] = {SB, SB + 1, SB + 2, SB + 3, SB + 4, SB + 5, SB + 6, SB + 7,
                                       SB + 8, SBB, SBB + 1, SBB + 2, SG, SG + 1, SG + 2, SG + 3,
                                       SG + 4, SG + 5, SALPHA, SBETA, SBETA + 1, SBETA + 2, SPHI, SK0};

// Outputs go to the sink in two halves: the global loads (the RK4 combine reads Q^n and the accumulator),
// issued together before the buffers of the outputs' slots are given up, and the stores, made while the
// next part is computed or copied.
// Right-hand side of the lane's cell of slab sl of the patch at qp.  Every lane of the
// work-group must call this (staging and barriers); only lanes with act = true compute.
template <typename T, int LOP, int XG, typename Sink>
__device__ __forceinline__ void rhs_slab_lds(const double *__restrict__ qp, double *lds, double *ldsb, int sl, bool act, uint32_t o0,
                                             const LdsCell<XG> &C0, const RhsParams &p, Sink &snk, const HaloSrc &hs)
{
    const Stager sg = lds_stager<XG>(qp, sl, hs);
    const PatchBuf qb{qp};
    const bool gdrv = p.shift != 0;
    const T sfac = gdrv ? T(1) : T(0);
    const T cc = cvt<T>(p.c);
    // the red terms of the Ghat equation (2 alpha gt^ik d_k tr At, with d_k gt^nm = -2 D_k^nm)
    // belong to the first-order formulation only
    const T red = p.formulation ? T(0) : T(1);
    // Round 3's Ghat sector shares the Ricci sector's loads and Christoffel symbols when the algebra is
    // FP32 (room in the register file); with FP64 algebra it reloads them in a block of its own, which
    // keeps the register peak of the Ricci sector down (four to twelve registers of a kernel spill; merged, 74).
    constexpr bool GHAT_IN_RICCI = sizeof(T) == 4;

    // carried between rounds
    T dtrA[3], sdBtr[3], GB[3], partD[3][6];
    double advkoAt[6], advkoB[9];
    T G1[3][3], H[3][3], U[3][3], E[6];
    T BB[3][3], curl[3][3];
    double rGb[3];
    // the pointwise parts of the gt, alpha, beta and phi equations, formed in round 3 where their
    // inputs are at hand (round 4 adds the Kreiss-Oliger sums and f b^i)
    double pwG[6], pwA, pwPhi;
    T bB[3];
    // Values of the cell that several rounds use, held in registers from round 1 on instead of read
    // again from memory in each round (the lines have left L2 by then: such reads were a third of a
    // stage's L2 misses).  With FP64 algebra the register file takes the shift, the metric, alpha and At
    // (a step on 4096 leaves: 16.19 -> 15.79 ms by the first two, 14.98 -> 14.79 ms by the others); with
    // the nine B too it spills.  With FP32 algebra B and D fit as well, as FP32 values (16.62 -> 15.28 ms).
    constexpr bool HOLD_ALL = sizeof(T) == 4;
    double be[3], gd0[6];  // loaded while round 1 is staged
    {
        const uint32_t o = fresh(o0);
#pragma unroll
        for (int k = 0; k < 3; ++k) be[k] = qb.load(o, SBETA + k);
#pragma unroll
        for (int k = 0; k < 6; ++k) gd0[k] = qb.load(o, SG + k);
    }
    T al0, At0[6], B0[9], D0[HOLD_ALL ? 18 : 1];
    auto held_metric = [&](double gd[6], double igd[6], double &detg, T g[6], T ig[6]) {
        load_metric_with<T>([&](int v) -> double { return fresh(gd0[v - SG]); }, gd, igd, detg, g, ig);
    };
    double ro2a[9], ro2b[6], ro3[20], ro4[24];  // each round's outputs, handed to the sink after the round

    // ------------------------------------------------------------ round 1: At, B
    const int rB[9] = {SB, SB + 1, SB + 2, SB + 3, SB + 4, SB + 5, SB + 6, SB + 7, SB + 8};
    const int rAt[6] = {SAT, SAT + 1, SAT + 2, SAT + 3, SAT + 4, SAT + 5};
    lds_issue(lds, rB, sg);
    lds_issue(ldsb, rAt, sg);
    wait_all_but(rAt);  // B has landed
    lds_swap();
    if (act) {
        {  // B: advection + KO, GB^i = gt^kl d_(k B_l)^i, sdBtr_k = d_(k B_l)^l, and the shift
           // terms of the D equations
            const LdsCell<XG> C = fresh(C0);
            double gd[6], igd[6], detg;
            T g[6], ig[6];
            held_metric(gd, igd, detg, g, ig);
            double dB[3][3][3];  // dB[l][i][k] = d_k B_l^i
#pragma unroll
            for (int i = 0; i < 3; ++i) GB[i] = sdBtr[i] = T(0);
            each_slot<9>(C, 0, [&](int n, const Points &q) {
                const SlotDeriv sd = stencils<LOP>(q, 0, be, p.advection);
                B0[n] = fresh(cvt<T>(q.own));
                keep(advkoB[n], gdrv ? sd.a + sd.k : 0.0);
#pragma unroll
                for (int k = 0; k < 3; ++k) keep(dB[n / 3][n % 3][k], sd.d[k]);
            });
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int l = 0; l < 3; ++l)
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        const T v = cvt<T>(dB[l][i][k]);
                        GB[i] += ig[sym(k, l)] * v;
                        if (i == l) sdBtr[k] += T(0.5) * v;
                        if (i == k) sdBtr[l] += T(0.5) * v;
                    }
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                T Y[3][3];  // d_k B_j^m + d_j B_k^m
#pragma unroll
                for (int j = 0; j < 3; ++j)
#pragma unroll
                    for (int m = 0; m < 3; ++m) Y[j][m] = cvt<T>(dB[j][m][k] + dB[k][m][j]);
                const T sdB = T(0.5) * (Y[0][0] + Y[1][1] + Y[2][2]);
#pragma unroll
                for (int i = 0; i < 3; ++i)
#pragma unroll
                    for (int j = i; j < 3; ++j) {
                        const int ij = sym(i, j);
                        T sb = T(0);
#pragma unroll
                        for (int m = 0; m < 3; ++m) sb += g[sym(m, i)] * Y[j][m] + g[sym(m, j)] * Y[i][m];
                        partD[k][ij] = sfac * (T(0.25) * sb - T(1.0 / 3.0) * g[ij] * sdB);
                    }
            }
        }
    }
    wait_memory<0>();  // At has landed
    lds_swap();
    const int rDa[9] = {SD, SD + 1, SD + 2, SD + 3, SD + 4, SD + 5, SD + 6, SD + 7, SD + 8};
    lds_issue(lds, rDa, sg);
    if (act) {
        {  // At: advection + KO, d_k tr(At), and the rest of the D equations
            const LdsCell<XG> C = fresh(C0);
            const uint32_t o = fresh(o0);
            auto q = [&](int v) -> double { return pw<1>(qb, o, C, v); };
            double dA[6][3];
            each_slot<6>(C, LDS_NA, [&](int s, const Points &q) {
                const SlotDeriv sd = stencils<LOP>(q, 0, be, p.advection);
                keep(advkoAt[s], sd.a + sd.k);
#pragma unroll
                for (int k = 0; k < 3; ++k) keep(dA[s][k], sd.d[k]);
            });
            double gd[6], igd[6], detg;
            T g[6], ig[6];
            held_metric(gd, igd, detg, g, ig);
            T At[6], D[3][6], Bm[3][3], A[3];
#pragma unroll
            for (int s = 0; s < 6; ++s) At[s] = cvt<T>(q(SAT + s));
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                A[k] = cvt<T>(q(SA + k));
#pragma unroll
                for (int s = 0; s < 6; ++s) D[k][s] = cvt<T>(q(SD + 6 * k + s));
#pragma unroll
                for (int i = 0; i < 3; ++i) Bm[k][i] = fresh(B0[3 * k + i]);
            }
            const T trB = Bm[0][0] + Bm[1][1] + Bm[2][2];
            const T trAt = tr6(ig, At);
            const T al = cvt<T>(q(SALPHA));
            al0 = fresh(al);
#pragma unroll
            for (int s = 0; s < 6; ++s) At0[s] = fresh(At[s]);
            if constexpr (HOLD_ALL) {
#pragma unroll
                for (int k = 0; k < 3; ++k) {
#pragma unroll
                    for (int s = 0; s < 6; ++s) D0[6 * k + s] = fresh(D[k][s]);
                }
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                T Dupk[6];
                {
                    T Dm[3][3];
#pragma unroll
                    for (int i = 0; i < 3; ++i)
#pragma unroll
                        for (int m = 0; m < 3; ++m)
                            Dm[i][m] = ig[sym(i, 0)] * D[k][sym(0, m)] + ig[sym(i, 1)] * D[k][sym(1, m)] +
                                       ig[sym(i, 2)] * D[k][sym(2, m)];
#pragma unroll
                    for (int i = 0; i < 3; ++i)
#pragma unroll
                        for (int j = i; j < 3; ++j)
                            Dupk[sym(i, j)] = Dm[i][0] * ig[sym(0, j)] + Dm[i][1] * ig[sym(1, j)] + Dm[i][2] * ig[sym(2, j)];
                }
                T dAk[6];
#pragma unroll
                for (int s = 0; s < 6; ++s) dAk[s] = cvt<T>(dA[s][k]);
                dtrA[k] = tr6(ig, dAk) - T(2) * tr6(At, Dupk);
#pragma unroll
                for (int i = 0; i < 3; ++i)
#pragma unroll
                    for (int j = i; j < 3; ++j) {
                        const int ij = sym(i, j);
                        T t = partD[k][ij];
                        t += -al * dAk[ij] + al * T(1.0 / 3.0) * g[ij] * dtrA[k];
#pragma unroll
                        for (int l = 0; l < 3; ++l)
                            t += Bm[k][l] * D[l][ij] + Bm[j][l] * D[k][sym(l, i)] + Bm[i][l] * D[k][sym(l, j)];
                        t += T(-2.0 / 3.0) * trB * D[k][ij];
                        t += -A[k] * (At[ij] - T(1.0 / 3.0) * g[ij] * trAt);
                        partD[k][ij] = t;
                    }
            }
        }
    }

    // ------------------------------------------------------------ round 2: D_x.., D_y.., D_zxx..D_zxz
    wait_memory<0>();
    lds_swap();
    const int rDb[6] = {SD + 9, SD + 10, SD + 11, SD + 12, SD + 13, SD + 14};
    lds_issue(ldsb, rDb, sg);
    auto D_slots = [&](auto first, auto count, double *out) {
        const LdsCell<XG> C = fresh(C0);
        double gd[6], igd[6], detg;
        T g[6], ig[6];
        held_metric(gd, igd, detg, g, ig);
        each_slot<count.value>(C, first.value, [&](int n, const Points &q) {
            const int j = first.value + n;
            const SlotDeriv sd = stencils<LOP>(q, 0, be, p.advection);
            dD_accumulate<T>(sd.d, j, ig, G1, H, U, E);
            keep(out[n], sd.a + static_cast<double>(partD[j / 6][j % 6]) + sd.k);
        });
    };
    if (act) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
#pragma unroll
            for (int j = 0; j < 3; ++j) G1[i][j] = H[i][j] = U[i][j] = T(0);
            E[i] = E[i + 3] = T(0);
        }
        D_slots(std::integral_constant<int, 0>{}, std::integral_constant<int, 9>{}, ro2a);
    }
    const int r2a[9] = {SD, SD + 1, SD + 2, SD + 3, SD + 4, SD + 5, SD + 6, SD + 7, SD + 8};
    const int r2b[6] = {SD + 9, SD + 10, SD + 11, SD + 12, SD + 13, SD + 14};
    double qa[9], qc[9], qb6[6], qd6[6];
    wait_memory<0>();
    if (act) snk.load(r2a, qa, qc, [&](int v) -> double { return pw<2>(qb, o0, C0, v); });
    lds_swap();
    const int r3a[9] = {SD + 15, SD + 16, SD + 17, SP, SP + 1, SP + 2, SA, SA + 1, SA + 2};
    lds_issue(lds, r3a, sg);
    if (act) D_slots(std::integral_constant<int, 9>{}, std::integral_constant<int, 6>{}, ro2b);
    wait_memory<0>();
    if (act) snk.load(r2b, qb6, qd6, [&](int v) -> double { return pw<2>(qb, o0, C0, v); });
    lds_swap();
    const int r3b[5] = {SGHAT, SGHAT + 1, SGHAT + 2, SK, STHETA};
    lds_issue(ldsb, r3b, sg);
    if (act) snk.store(r2a, ro2a, qa, qc);

    // ------------------------------------------------------------ round 3
    // buffers: 0..2 D_zyy, D_zyz, D_zzz; 3..5 P; 6..8 A; 9..11 Ghat; 12 K; 13 Theta
    if (act) {
        {
            const LdsCell<XG> C = fresh(C0);
            double gd[6], igd[6], detg;
            T g[6], ig[6];
            held_metric(gd, igd, detg, g, ig);
            each_slot<3>(C, 0, [&](int j, const Points &q) {
                const SlotDeriv sd = stencils<LOP>(q, 0, be, p.advection);
                dD_accumulate<T>(sd.d, 15 + j, ig, G1, H, U, E);
                keep(ro3[j], sd.a + static_cast<double>(partD[2][3 + j]) + sd.k);
            });
        }
        snk.store(r2b, ro2b, qb6, qd6);
    }
    wait_memory<0>();
    lds_swap();
    if (act) {
        const LdsCell<XG> C = fresh(C0);
        const uint32_t o = fresh(o0);
        {  // ---- Ricci sector: At, K, Theta; the curl term of B
            const uint32_t o1 = fresh(o);
            auto q1 = [&](int v) -> double { return pw<3>(qb, o1, C, v); };
            double gd[6], igd[6], detg;
            T g[6], ig[6];
            held_metric(gd, igd, detg, g, ig);
            const double phid = q1(SPHI), iphid = 1.0 / phid;
            double Pphid[3];
#pragma unroll
            for (int l = 0; l < 3; ++l) Pphid[l] = q1(SP + l) * iphid;
            T Pphi[3], Puphi[3], sdPphi[6];
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                Pphi[m] = cvt<T>(Pphid[m]);
                Puphi[m] = cvt<T>(igd[sym(m, 0)] * Pphid[0] + igd[sym(m, 1)] * Pphid[1] + igd[sym(m, 2)] * Pphid[2]);
            }
            {
                double dP[3][3];  // dP[j][i] = d_i P_j
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    const SlotDeriv sd = stencils(C, 3 + j);
#pragma unroll
                    for (int i = 0; i < 3; ++i) dP[j][i] = sd.d[i];
                }
#pragma unroll
                for (int i = 0; i < 3; ++i)
#pragma unroll
                    for (int j = i; j < 3; ++j) sdPphi[sym(i, j)] = cvt<T>(0.5 * (dP[j][i] + dP[i][j]) * iphid);
            }
            T D[3][6];
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int s = 0; s < 6; ++s) D[k][s] = HOLD_ALL ? fresh(D0[HOLD_ALL ? 6 * k + s : 0]) : cvt<T>(q1(SD + 6 * k + s));
            T Dup[3][6], Gl[3][6], Gt[3][6], Gtv[3];
            raise_D(ig, D, Dup);
            christoffel(ig, D, Gl, Gt, Gtv);
            T V[3], Wl[3];
#pragma unroll
            for (int l = 0; l < 3; ++l) {
                V[l] = Dup[0][sym(0, l)] + Dup[1][sym(1, l)] + Dup[2][sym(2, l)];
                Wl[l] = tr6(ig, Gl[l]);
            }
            T Gam[3][6];
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int i = 0; i < 3; ++i)
#pragma unroll
                    for (int j = i; j < 3; ++j) {
                        T t = -g[sym(i, j)] * Puphi[k];
                        if (k == i) t += Pphi[j];
                        if (k == j) t += Pphi[i];
                        Gam[k][sym(i, j)] = Gt[k][sym(i, j)] - t;
                    }
            T Gc[3];
#pragma unroll
            for (int l = 0; l < 3; ++l) Gc[l] = Gam[0][sym(l, 0)] + Gam[1][sym(l, 1)] + Gam[2][sym(l, 2)];
            const T PP = Pphi[0] * Puphi[0] + Pphi[1] * Puphi[1] + Pphi[2] * Puphi[2];
            const T VP = V[0] * Pphi[0] + V[1] * Pphi[1] + V[2] * Pphi[2];
            const T trsdP = tr6(ig, sdPphi);
            T Ric[6];
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int j = i; j < 3; ++j) {
                    const int ij = sym(i, j);
                    T s1 = T(-2) * (V[0] * Gl[0][ij] + V[1] * Gl[1][ij] + V[2] * Gl[2][ij]);
                    s1 += T(0.5) * (G1[i][j] + H[i][j] + G1[j][i] + H[j][i]) - E[ij];
                    s1 += T(2) * (D[0][ij] * Puphi[0] + D[1][ij] * Puphi[1] + D[2][ij] * Puphi[2] - g[ij] * VP);
                    s1 += -(T(2) * sdPphi[ij] - g[ij] * trsdP);
                    s1 += T(2) * Pphi[i] * Pphi[j] - g[ij] * PP;
                    T DD = T(0);
#pragma unroll
                    for (int s = 0; s < 6; ++s) DD += (s == 0 || s == 3 || s == 5 ? T(1) : T(2)) * Dup[j][s] * D[i][s];
                    const T s2 =
                        T(-2) * DD + T(0.5) * (U[j][i] + U[i][j]) - T(3) * sdPphi[ij] + T(3) * Pphi[i] * Pphi[j];
                    T gg = Gam[0][ij] * Gc[0] + Gam[1][ij] * Gc[1] + Gam[2][ij] * Gc[2];
#pragma unroll
                    for (int l = 0; l < 3; ++l)
#pragma unroll
                        for (int m = 0; m < 3; ++m) gg -= Gam[l][sym(i, m)] * Gam[m][sym(l, j)];
                    Ric[ij] = s1 - s2 + gg;
                }
            T dGt[3][3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                T F[3];
#pragma unroll
                for (int n = 0; n < 3; ++n) F[n] = H[k][n] + G1[k][n] - T(0.5) * (U[k][n] + U[n][k]);
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    T t = T(0);
#pragma unroll
                    for (int s = 0; s < 6; ++s) t += (s == 0 || s == 3 || s == 5 ? T(1) : T(2)) * Dup[k][s] * Gt[i][s];
                    t = T(-2) * t -
                        T(2) * (Dup[k][sym(i, 0)] * Wl[0] + Dup[k][sym(i, 1)] * Wl[1] + Dup[k][sym(i, 2)] * Wl[2]);
                    dGt[k][i] = t + ig[sym(i, 0)] * F[0] + ig[sym(i, 1)] * F[1] + ig[sym(i, 2)] * F[2];
                }
            }
            T dG[3], Zl[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) dG[i] = cvt<T>(q1(SGHAT + i)) - Gtv[i];
#pragma unroll
            for (int i = 0; i < 3; ++i)
                Zl[i] = T(0.5) * (g[sym(i, 0)] * dG[0] + g[sym(i, 1)] * dG[1] + g[sym(i, 2)] * dG[2]);
            T RZ[6];
            {
                T nZ[3][3];
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    T dGh[3];
#pragma unroll
                    for (int l = 0; l < 3; ++l) dGh[l] = cvt<T>(fd(C, 9 + l, i)) - dGt[i][l];
#pragma unroll
                    for (int j = 0; j < 3; ++j) {
                        T t = D[i][sym(j, 0)] * dG[0] + D[i][sym(j, 1)] * dG[1] + D[i][sym(j, 2)] * dG[2];
#pragma unroll
                        for (int l = 0; l < 3; ++l) t += T(0.5) * g[sym(j, l)] * dGh[l] - Gam[l][sym(i, j)] * Zl[l];
                        nZ[i][j] = t;
                    }
                }
#pragma unroll
                for (int i = 0; i < 3; ++i)
#pragma unroll
                    for (int j = i; j < 3; ++j) RZ[sym(i, j)] = Ric[sym(i, j)] + nZ[i][j] + nZ[j][i];
            }
            T A[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) A[k] = cvt<T>(q1(SA + k));
            T DDa[6];
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int j = i; j < 3; ++j)
                    DDa[sym(i, j)] = T(0.5) * cvt<T>(fd(C, 6 + j, i) + fd(C, 6 + i, j)) -
                                     (Gam[0][sym(i, j)] * A[0] + Gam[1][sym(i, j)] * A[1] + Gam[2][sym(i, j)] * A[2]);
            const T al = fresh(al0), Kt = cvt<T>(q1(SK)), Th = cvt<T>(q1(STHETA));
            T X[6];
#pragma unroll
            for (int s = 0; s < 6; ++s) X[s] = -DDa[s] + al * RZ[s];
            const T trX = tr6(ig, X);
            const T phi2 = cvt<T>(phid * phid);
            const T RpZ = phi2 * tr6(ig, RZ);
            const T lapal = phi2 * tr6(ig, DDa);
            T At[6];
#pragma unroll
            for (int s = 0; s < 6; ++s) At[s] = fresh(At0[s]);
            T Am[3][3];
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int j = 0; j < 3; ++j)
                    Am[i][j] = ig[sym(i, 0)] * At[sym(0, j)] + ig[sym(i, 1)] * At[sym(1, j)] + ig[sym(i, 2)] * At[sym(2, j)];
            T AA = T(0);
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int j = 0; j < 3; ++j) AA += Am[i][j] * Am[j][i];
            T Bm[3][3];
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int i = 0; i < 3; ++i) Bm[k][i] = HOLD_ALL ? fresh(B0[HOLD_ALL ? 3 * k + i : 0]) : cvt<T>(q1(SB + 3 * k + i));
            const T trB = Bm[0][0] + Bm[1][1] + Bm[2][2];
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int j = i; j < 3; ++j) {
                    const int ij = sym(i, j);
                    T t = T(0);
#pragma unroll
                    for (int k = 0; k < 3; ++k) t += At[sym(k, i)] * Bm[j][k] + At[sym(k, j)] * Bm[i][k];
                    t += T(-2.0 / 3.0) * At[ij] * trB;
                    t += al * At[ij] * (Kt - T(2) * Th * cc);
                    t += T(-2) * al * (At[sym(i, 0)] * Am[0][j] + At[sym(i, 1)] * Am[1][j] + At[sym(i, 2)] * Am[2][j]);
                    const T tf = X[ij] - T(1.0 / 3.0) * g[ij] * trX;
                    keep(ro3[3 + ij], advkoAt[ij] + static_cast<double>(t) + phid * phid * static_cast<double>(tf));
                }
            const T kap1 = cvt<T>(p.kappa1), kap2 = cvt<T>(p.kappa2);
            CCZ4_PHASE_BARRIER();
            const SlotDeriv sK = stencils<LOP>(C, 12, be, p.advection);
            keep(ro3[9], (sK.a + static_cast<double>(-lapal + al * RpZ + al * Kt * (Kt - T(2) * Th * cc) -
                                                             T(3) * al * kap1 * (T(1) + kap2) * Th) +
                      sK.k));
            const T ee2 = cvt<T>(p.e * p.e);
            const T ZA = T(0.5) * phi2 * (dG[0] * A[0] + dG[1] * A[1] + dG[2] * A[2]);
            const SlotDeriv sTh = stencils<LOP>(C, 13, be, p.advection);
            keep(ro3[10], (sTh.a +
                                static_cast<double>(T(0.5) * al * ee2 * (RpZ + T(2.0 / 3.0) * Kt * Kt - AA) -
                                                    al * Th * Kt * cc - ZA - al * kap1 * (T(2) + kap2) * Th) +
                      sTh.k));
            // B without f d_k b^i (completed in round 4): B_k^l B_l^i and alpha^2 mu gt^ij (curl D - curl P)
            if (gdrv) {
                T cP[3][3];
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    cP[k][k] = T(0);
#pragma unroll
                    for (int j = k + 1; j < 3; ++j) {
                        const double wv = (fd(C, 3 + j, k) - fd(C, 3 + k, j)) * iphid;
                        cP[k][j] = cvt<T>(wv);
                        cP[j][k] = cvt<T>(-wv);
                    }
                }
                const T a2mu = al * al * cvt<T>(p.mu);
#pragma unroll
                for (int k = 0; k < 3; ++k)
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        BB[k][i] = Bm[k][0] * Bm[0][i] + Bm[k][1] * Bm[1][i] + Bm[k][2] * Bm[2][i];
                        T cu = T(0);
#pragma unroll
                        for (int j = 0; j < 3; ++j) cu += ig[sym(i, j)] * ((H[k][j] - G1[k][j]) - cP[k][j]);
                        curl[k][i] = a2mu * cu;
                    }
            }
            if constexpr (GHAT_IN_RICCI)  // the same metric, D, At, B, A, P / phi and Christoffel symbols
                ghat_sector<T, LOP, XG>(C, p, be, g, ig, gd, detg, D, Gt, Gtv, At, Am, Bm, A, Pphi, trB, al, Kt, Th, Zl, GB,
                                    sdBtr, dtrA, red, sfac, ro3, rGb, pwG);
        }
        CCZ4_PHASE_BARRIER();
        if constexpr (!GHAT_IN_RICCI) {  // ---- Ghat^i, and the part of b^i it shares
            const uint32_t o1 = fresh(o);
            auto q1 = [&](int v) -> double { return pw<3>(qb, o1, C, v); };
            double gd[6], igd[6], detg;
            T g[6], ig[6];
            held_metric(gd, igd, detg, g, ig);
            T D[3][6], At[6];
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int s = 0; s < 6; ++s) D[k][s] = HOLD_ALL ? fresh(D0[HOLD_ALL ? 6 * k + s : 0]) : cvt<T>(q1(SD + 6 * k + s));
#pragma unroll
            for (int s = 0; s < 6; ++s) At[s] = fresh(At0[s]);
            T Dup[3][6], Gl[3][6], Gt[3][6], Gtv[3];
            raise_D(ig, D, Dup);
            christoffel(ig, D, Gl, Gt, Gtv);
            T Am[3][3];
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int j = 0; j < 3; ++j)
                    Am[i][j] = ig[sym(i, 0)] * At[sym(0, j)] + ig[sym(i, 1)] * At[sym(1, j)] + ig[sym(i, 2)] * At[sym(2, j)];
            T Bm[3][3], A[3], Ph[3];
            const double iphid = 1.0 / q1(SPHI);
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                A[k] = cvt<T>(q1(SA + k));
                Ph[k] = cvt<T>(q1(SP + k) * iphid);
#pragma unroll
                for (int i = 0; i < 3; ++i) Bm[k][i] = HOLD_ALL ? fresh(B0[HOLD_ALL ? 3 * k + i : 0]) : cvt<T>(q1(SB + 3 * k + i));
            }
            const T trB = Bm[0][0] + Bm[1][1] + Bm[2][2];
            const T al = fresh(al0), Kt = cvt<T>(q1(SK)), Th = cvt<T>(q1(STHETA));
            T dG[3], Zl[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) dG[i] = cvt<T>(q1(SGHAT + i)) - Gtv[i];
#pragma unroll
            for (int i = 0; i < 3; ++i)
                Zl[i] = T(0.5) * (g[sym(i, 0)] * dG[0] + g[sym(i, 1)] * dG[1] + g[sym(i, 2)] * dG[2]);
            ghat_sector<T, LOP, XG>(C, p, be, g, ig, gd, detg, D, Gt, Gtv, At, Am, Bm, A, Ph, trB, al, Kt, Th, Zl, GB, sdBtr,
                                dtrA, red, sfac, ro3, rGb, pwG);
        }
        CCZ4_PHASE_BARRIER();
        {  // ---- A_k and P_k
            const uint32_t o1 = fresh(o);
            auto q1 = [&](int v) -> double { return pw<3>(qb, o1, C, v); };
            T Bm[3][3], A[3], P[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                A[k] = cvt<T>(q1(SA + k));
                P[k] = cvt<T>(q1(SP + k));
#pragma unroll
                for (int i = 0; i < 3; ++i) Bm[k][i] = HOLD_ALL ? fresh(B0[HOLD_ALL ? 3 * k + i : 0]) : cvt<T>(q1(SB + 3 * k + i));
            }
            const T trB = Bm[0][0] + Bm[1][1] + Bm[2][2];
            const T al = fresh(al0), Kt = cvt<T>(q1(SK)), Th = cvt<T>(q1(STHETA)), K0 = cvt<T>(q1(SK0));
            const double phid = q1(SPHI);
            const bool onelog = p.slicing == 1;
            const T ga = onelog ? T(2) / al : T(1);
            const T ga_lin = onelog ? T(2) : T(2) * al;  // 2 alpha g + alpha^2 g'
            const T theta_term = Kt - K0 - T(2) * cc * Th;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const T dK = cvt<T>(fd(C, 12, k)), dTh = cvt<T>(fd(C, 13, k));
                T t = -al * al * ga * (dK - T(2) * cc * dTh) - al * ga * dtrA[k];
                t += Bm[k][0] * A[0] + Bm[k][1] * A[1] + Bm[k][2] * A[2];
                t += -ga_lin * theta_term * A[k];
                const SlotDeriv sA = stencils<LOP>(C, 6 + k, be, p.advection);
                keep(ro3[14 + k], sA.a + static_cast<double>(t) + sA.k);
                const T u = Bm[k][0] * P[0] + Bm[k][1] * P[1] + Bm[k][2] * P[2] + T(1.0 / 3.0) * (al * Kt - trB) * P[k];
                const T phipart =
                    T(1.0 / 3.0) * (al * dK - sdBtr[k]) + T(1.0 / 3.0) * al * dtrA[k] + T(1.0 / 3.0) * Kt * A[k];
                const SlotDeriv sP = stencils<LOP>(C, 3 + k, be, p.advection);
                keep(ro3[17 + k], sP.a + static_cast<double>(u) + phid * static_cast<double>(phipart) + sP.k);
            }
            // alpha: beta^k A_k - alpha^2 g (K - K_0 - 2 c Theta); beta^i: beta^k B_k^i (+ f b^i in round 4);
            // phi: beta^k P_k + phi (alpha K - tr B) / 3
            T bet[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) bet[k] = cvt<T>(be[k]);
            keep(pwA, static_cast<double>(bet[0] * A[0] + bet[1] * A[1] + bet[2] * A[2] -
                                          al * al * ga * (Kt - K0 - T(2) * cc * Th)));
#pragma unroll
            for (int i = 0; i < 3; ++i) bB[i] = bet[0] * Bm[0][i] + bet[1] * Bm[1][i] + bet[2] * Bm[2][i];
            keep(pwPhi, be[0] * q1(SP) + be[1] * q1(SP + 1) + be[2] * q1(SP + 2) +
                            phid * static_cast<double>((al * Kt - trB) * T(1.0 / 3.0)));
        }
    }

    {
        const int r4a[9] = {SBB, SBB + 1, SBB + 2, SG, SG + 1, SG + 2, SG + 3, SG + 4, SG + 5};
        const int r4b[5] = {SALPHA, SBETA, SBETA + 1, SBETA + 2, SPHI};
        double qa3[20], qc3[20];
        if (act)
            snk.load(R3_OUT, qa3, qc3, [&](int v) -> double {
                if (sizeof(T) == 8 && v >= SAT && v < SAT + 6) return static_cast<double>(At0[v - SAT]);
                return pw<3>(qb, o0, C0, v);
            });
        lds_swap();
        lds_issue(lds, r4a, sg);
        lds_issue(ldsb, r4b, sg);
        wait_all_but(r4b);
        if (act) snk.store(R3_OUT, ro3, qa3, qc3);
    }
    lds_swap();

    // ------------------------------------------------------------ round 4
    // buffers: 0..2 b; 3..8 gt; 9 alpha; 10..12 beta; 13 phi
    if (act) {
        const LdsCell<XG> C = fresh(C0);
        // B_k^i and b^i
        if (gdrv) {
            const T ff = cvt<T>(p.f);
            each_slot<3>(C, 0, [&](int i, const Points &pt) {
                const SlotDeriv sb = stencils<LOP>(pt, 0, be, p.advection);
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    T t = ff * cvt<T>(sb.d[k]);
                    t += BB[k][i];
                    t += curl[k][i];
                    keep(ro4[3 * k + i], advkoB[3 * k + i] + static_cast<double>(t));
                }
                keep(ro4[9 + i], rGb[i] + sb.a - p.eta * pt.own + sb.k);
            });
        } else {
#pragma unroll
            for (int s = 0; s < 9; ++s) keep(ro4[s], 0.0);
#pragma unroll
            for (int i = 0; i < 3; ++i) keep(ro4[9 + i], 0.0);
        }
        // gt_ij, alpha, beta^i, phi: the pointwise parts from round 3 and the KO sums; K_0: 0
        each_slot<6>(C, 3, [&](int s, const Points &pt) { keep(ro4[12 + s], pwG[s] + ko(pt, 0)); });
    }
    wait_memory<0>();
    lds_swap();
    if (act) {
        const LdsCell<XG> C = fresh(C0);
        const uint32_t o = fresh(o0);
        auto q = [&](int v) -> double { return pw<4>(qb, o, C, v); };
        each_slot<5>(C, LDS_NA, [&](int n, const Points &pt) {
            const double k = ko(pt, 0);
            if (n == 0) keep(ro4[18], pwA + k);
            else if (n == 4) keep(ro4[22], pwPhi + k);
            else if (gdrv) keep(ro4[18 + n], static_cast<double>(bB[n - 1] + cvt<T>(p.f) * cvt<T>(q(SBB + n - 1))) + k);
            else keep(ro4[18 + n], 0.0);
        });
        keep(ro4[23], 0.0);
    }
    {
        double qa[24], qc[24];
        if (act) {
            snk.load(R4_OUT, qa, qc, [&](int v) -> double { return pw<4>(qb, o0, C0, v); });
            snk.store(R4_OUT, ro4, qa, qc);
        }
    }
    if (act) snk.finish();
}

}  // namespace ccz4
