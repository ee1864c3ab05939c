// Learned refinement indicator on gfx950: per-patch features, a 81 -> 64 -> 64 -> 3 perceptron
// on BF16 matrix cores (v_mfma_f32_16x16x16_bf16, FP32 accumulation) with its loss gradient,
// an Adam step on FP32 master weights, and the combination with the plain criterion.
//
// Parameter vector (NPARAM = 9603 floats), row-major, out x in:
//   W1[64][81] b1[64] W2[64][64] b2[64] W3[3][64] b3[3]
// The inputs are standardised in FP32, x = (feat - mu) * inv_sigma, then rounded to BF16 with
// the weights; hidden activations are rounded to BF16 after the ReLU; in the backward pass the
// pre-activation gradients entering a product are rounded to BF16 and the roundings are taken
// as the identity (straight-through).  The bias gradients sum the FP32 gradients.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>

#include "ccz4_kernels.hpp"
#include "ccz4_mlp.hpp"

namespace ccz4 {

namespace {

constexpr int NIN = MLP_NIN, NINP = 96, NH = MLP_NH, NOUT = MLP_NOUT, NOUTP = 16;
constexpr int OW1 = 0, OB1 = OW1 + NH * NIN, OW2 = OB1 + NH, OB2 = OW2 + NH * NH, OW3 = OB2 + NH,
              OB3 = OW3 + NOUT * NH;
static_assert(OB3 + NOUT == MLP_NPARAM, "parameter layout");
constexpr int TILE = 64;  // rows (patches) of a forward work-group's four waves; the unit of the workspace

typedef short bf4_t __attribute__((ext_vector_type(4)));
typedef float f4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bfv4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// FP32 -> BF16, round to nearest, ties to even
__device__ __forceinline__ bf4_t pack4(f4_t v) { return __builtin_bit_cast(bf4_t, __builtin_convertvector(v, bfv4_t)); }

__device__ __forceinline__ f4_t mma(bf4_t a, bf4_t b, f4_t c)
{
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// Every product runs on one wave's 16 rows with the rows as columns: Z^T = W X^T.  Of a 16 x 16 x 16
// product lane l (li = l % 16, g = l / 16) supplies A(li, 4 g + r) and B(4 g + r, li), r = 0..3, and
// holds C(4 g + r, li): unit 16 t + 4 g + r of row li, tile t.  That is the B operand of the next
// layer's k-chunk t, so the activations and the back-propagated gradients go from product to product
// in registers, without LDS and without a barrier; the weights are A operands held in registers for
// all the rows of a wave.  (One work-group per 64 rows with every operand gathered from LDS two bytes
// at a time, the weights converted again for each, took 45 and 382 us forward for 20,112 and 241,344
// rows; now 12 and 38 us.)
struct MlpWeights {
    bf4_t w1[4][6], w2[4][4], w3[4];  // [tile of 16 units][chunk of 16 inputs]
    __device__ __forceinline__ bf4_t f1(int t, int c) const { return w1[t][c]; }
    __device__ __forceinline__ bf4_t f2(int t, int c) const { return w2[t][c]; }
    __device__ __forceinline__ bf4_t f3(int t) const { return w3[t]; }
};

// (clamped indices and selects: no branch per element)
__device__ __forceinline__ bf4_t weight_frag(const float *__restrict__ w, int row, int rows, int col, int cols)
{
    f4_t v;
    const float *p = w + (row < rows ? row : 0) * cols;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float t = p[col + r < cols ? col + r : 0];
        v[r] = row < rows && col + r < cols ? t : 0.f;
    }
    return pack4(v);
}

__device__ __forceinline__ void load_weights(MlpWeights &W, const float *__restrict__ prm, int li, int g)
{
#pragma unroll
    for (int t = 0; t < 4; ++t) {
#pragma unroll
        for (int c = 0; c < 6; ++c) W.w1[t][c] = weight_frag(prm + OW1, 16 * t + li, NH, 16 * c + 4 * g, NIN);
#pragma unroll
        for (int c = 0; c < 4; ++c) W.w2[t][c] = weight_frag(prm + OW2, 16 * t + li, NH, 16 * c + 4 * g, NH);
        W.w3[t] = weight_frag(prm + OW3, li, NOUT, 16 * t + 4 * g, NH);
    }
}

// The vectors that every row uses, zero where padded: normalisation and biases.  Read four at a time (vec4),
// at multiples of 16 bytes.
struct alignas(16) MlpVectors {
    float mu[NINP], is[NINP], b1[NH], b2[NH], b3[NOUTP];
};
static_assert(NINP % 4 == 0 && NH % 4 == 0 && NOUTP % 4 == 0, "whole groups of four");

__device__ __forceinline__ void load_vectors(MlpVectors &V, const float *__restrict__ prm, const float *__restrict__ norm)
{
    for (int i = threadIdx.x; i < NINP; i += blockDim.x) {
        V.mu[i] = i < NIN ? norm[i] : 0.f;
        V.is[i] = i < NIN ? norm[NIN + i] : 0.f;
        if (i < NH) {
            V.b1[i] = prm[OB1 + i];
            V.b2[i] = prm[OB2 + i];
        }
        if (i < NOUTP) V.b3[i] = i < NOUT ? prm[OB3 + i] : 0.f;
    }
    __syncthreads();
}

__device__ __forceinline__ f4_t vec4(const float *v) { return *reinterpret_cast<const f4_t *>(v); }

// One row's features as loaded: chunk c holds inputs 16 c + 4 g + r (a row is 81 floats: four-byte
// aligned), zero beyond the last input or row.
struct MlpRow {
    f4_t f[6];
};

__device__ __forceinline__ MlpRow load_row(const float *__restrict__ feat, int64_t row, int64_t n, int g)
{
    MlpRow R;
    const bool in = row < n;
    const float *f = feat + (in ? row : 0) * NIN + 4 * g;
#pragma unroll
    for (int c = 0; c < 5; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) R.f[c][r] = in ? f[16 * c + r] : 0.f;
    R.f[5] = f4_t{in && g == 0 ? f[80] : 0.f, 0.f, 0.f, 0.f};
    return R;
}

// The standardised inputs, x = (feat - mu) * inv_sigma in FP32, then BF16; zero rows beyond n.
__device__ __forceinline__ void standardise(const MlpVectors &V, const MlpRow &R, bool in, int g, bf4_t x[6])
{
#pragma unroll
    for (int c = 0; c < 6; ++c) {
        const f4_t mu = vec4(V.mu + 16 * c + 4 * g), is = vec4(V.is + 16 * c + 4 * g);
        f4_t v;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma clang fp contract(off)
            const float d = R.f[c][r] - mu[r];
            v[r] = in ? d * is[r] : 0.f;
        }
        x[c] = pack4(v);
    }
}

__device__ __forceinline__ f4_t relu4(f4_t z)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) z[r] = z[r] > 0.f ? z[r] : 0.f;
    return z;
}

// z1, z2 (pre-activations), a1, a2 (BF16 activations) and z3 (logits of row li: classes r = 0..2 of the
// lanes g = 0)
template <typename Weights>
__device__ __forceinline__ void mlp_layers(const Weights &W, const MlpVectors &V, int g, const bf4_t x[6], f4_t z1[4],
                                           bf4_t a1[4], f4_t z2[4], bf4_t a2[4], f4_t &z3)
{
#pragma unroll
    for (int t = 0; t < 4; ++t) z1[t] = f4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < 6; ++c)
#pragma unroll
        for (int t = 0; t < 4; ++t) z1[t] = mma(W.f1(t, c), x[c], z1[t]);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        z1[t] += vec4(V.b1 + 16 * t + 4 * g);
        a1[t] = pack4(relu4(z1[t]));
        z2[t] = f4_t{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int t = 0; t < 4; ++t) z2[t] = mma(W.f2(t, c), a1[c], z2[t]);
    z3 = f4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        z2[t] += vec4(V.b2 + 16 * t + 4 * g);
        a2[t] = pack4(relu4(z2[t]));
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) z3 = mma(W.f3(t), a2[t], z3);
    z3 += vec4(V.b3 + 4 * g);
}

// Waves take blocks of 16 rows in turn, the next block's features in flight meanwhile.
__global__ __launch_bounds__(256) void k_mlp_forward(const float *__restrict__ prm, const float *__restrict__ norm,
                                                     const float *__restrict__ feat, int64_t n,
                                                     float *__restrict__ logits)
{
    __shared__ MlpVectors V;
    const int l = threadIdx.x & 63, li = l & 15, g = l >> 4;
    const int64_t waves = (int64_t)gridDim.x * 4, first = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    MlpRow next = load_row(feat, first * 16 + li, n, g);
    MlpWeights W;
    load_weights(W, prm, li, g);
    load_vectors(V, prm, norm);
    for (int64_t b = first; b * 16 < n; b += waves) {
        const int64_t row = b * 16 + li;
        const MlpRow R = next;
        next = load_row(feat, row + waves * 16, n, g);
        bf4_t x[6], a1[4], a2[4];
        f4_t z1[4], z2[4], z3;
        standardise(V, R, row < n, g, x);
        mlp_layers(W, V, g, x, z1, a1, z2, a2, z3);
        if (g == 0 && row < n)
#pragma unroll
            for (int j = 0; j < NOUT; ++j) logits[row * NOUT + j] = z3[j];
    }
}

// Rows of one pass of a gradient work-group: 16 for each of its eight waves.
constexpr int GROWS = 128, GWAVES = 8;
// The operands of the weight gradients (products over the rows) in LDS, unit by unit with the rows
// contiguous: a lane writes its 4 x 1 piece of a block and reads four rows of one unit.  The row pitch
// of 132 spreads the units that a read touches over the banks.
constexpr int GPITCH = 132;
struct MlpOperands {
    uint16_t x[NINP][GPITCH], a1[NH][GPITCH], a2[NH][GPITCH], d1[NH][GPITCH], d2[NH][GPITCH], d3[NOUTP][GPITCH];
};

__device__ __forceinline__ void put_block(uint16_t (*u)[GPITCH], int unit, int row, bf4_t v)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) u[unit + r][row] = (uint16_t)v[r];
}

__device__ __forceinline__ bf4_t get_block(const uint16_t (*u)[GPITCH], int unit, int row)
{
    return *reinterpret_cast<const bf4_t *>(&u[unit][row]);
}

// The weights as operands in LDS, one fragment of 64 lanes each (a gradient wave's registers hold its
// share of the gradients instead), and those of the backward pass, W2^T and W3^T.
struct MlpFragments {
    bf4_t w1[4][6][64], w2[4][4][64], w3[4][64], w2t[4][4][64], w3t[4][64];
};
struct MlpLdsWeights {
    const MlpFragments &F;
    int l;
    __device__ __forceinline__ bf4_t f1(int t, int c) const { return F.w1[t][c][l]; }
    __device__ __forceinline__ bf4_t f2(int t, int c) const { return F.w2[t][c][l]; }
    __device__ __forceinline__ bf4_t f3(int t) const { return F.w3[t][l]; }
};

// wave w of eight fills its share: tile w % 4 of everything, split by w / 4
__device__ __forceinline__ void load_fragments(MlpFragments &F, const float *__restrict__ prm, int w, int l)
{
    const int li = l & 15, g = l >> 4, t = w & 3;
    if (w < 4) {
#pragma unroll
        for (int c = 0; c < 6; ++c) F.w1[t][c][l] = weight_frag(prm + OW1, 16 * t + li, NH, 16 * c + 4 * g, NIN);
        F.w3[t][l] = weight_frag(prm + OW3, li, NOUT, 16 * t + 4 * g, NH);
    } else {
        f4_t v;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            F.w2[t][c][l] = weight_frag(prm + OW2, 16 * t + li, NH, 16 * c + 4 * g, NH);
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = prm[OW2 + (16 * c + 4 * g + r) * NH + 16 * t + li];
            F.w2t[t][c][l] = pack4(v);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float u = prm[OW3 + (r < NOUT ? r : 0) * NH + 16 * t + li];
            v[r] = g == 0 && r < NOUT ? u : 0.f;
        }
        F.w3t[t][l] = pack4(v);
    }
}

// Loss and gradient sums of a work-group's rows: part[blk][0 .. NPARAM-1] gradient, [NPARAM] loss sum.
// Each wave takes 16 of a pass's 128 rows through the layers and back in registers; the gradients of
// the weights are products over the rows, whose operands pass through LDS once.  The 44 tiles of 16 x
// 16 of the weight gradients are shared out: wave w holds tile row w / 2 of W1 and W2 (the column tiles
// of half w % 2) and, for even w, tile w / 2 of W3, in registers over all passes, so that no sum is
// taken across waves and a launch leaves at most MLP_GRAD_BLOCKS partials (before, one for every 64
// rows: 145 MB written and read again for 241,344 rows).  Two waves per SIMD: the layers are chains of
// dependent products, bound by their latency.  Gradient and reduction of 27 / 4096 / 241,344 rows:
// 33 / 50 / 559 us with operands gathered element by element, 14 / 17 / 62 us now (109 us with one
// wave per SIMD that holds all gradients, 113 us with the weights in registers, which then spill).
// With trace != nullptr, each row also leaves the operands of its matrix products there (as FP32
// values, MLP_TRACE per row): the BF16 standardised input, the BF16 activations a1 and a2, and the
// FP32 pre-activation gradients d3, d2 and d1 before their BF16 rounding.
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_mlp_grad(
    const float *__restrict__ prm, const float *__restrict__ norm, const float *__restrict__ feat,
    const int8_t *__restrict__ tags, int64_t n, float *__restrict__ part, float *__restrict__ trace)
{
    __shared__ MlpVectors V;
    __shared__ __align__(16) MlpOperands S;
    __shared__ MlpFragments F;
    __shared__ float bias[GWAVES][2 * NH + NOUT + 1];
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), l = threadIdx.x & 63, li = l & 15, g = l >> 4;
    const int64_t stride = (int64_t)gridDim.x * GROWS, first = (int64_t)blockIdx.x * GROWS + 16 * w + li;
    MlpRow next = load_row(feat, first, n, g);
    int next_tag = first < n ? tags[first] : 0;
    load_fragments(F, prm, w, l);
    const MlpLdsWeights W{F, l};
    load_vectors(V, prm, norm);  // with a barrier
    const f4_t zero = {0.f, 0.f, 0.f, 0.f};
    const int ot = w >> 1, half = w & 1;
    // the sums of a pass's two halves of 64 rows apart: half as long, each, as one chain over all of them (which on
    // 65..190 rows had up to 1.2 times the rounding of sums of 64 rows)
    f4_t gw1[2][3], gw2[2][2], gw3[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int c = 0; c < 3; ++c) gw1[h][c] = zero;
#pragma unroll
        for (int c = 0; c < 2; ++c) gw2[h][c] = zero;
        gw3[h] = zero;
    }
    f4_t gb1[4] = {zero, zero, zero, zero}, gb2[4] = {zero, zero, zero, zero}, gb3 = zero;
    float loss = 0.f;
    const float inv_n = 1.0f / (float)n;
    for (int64_t b = (int64_t)blockIdx.x * GROWS; b < n; b += stride) {
        const int64_t row = b + 16 * w + li;
        const bool in = row < n;
        const MlpRow R = next;
        const int lab = next_tag + 1;  // COARSEN, KEEP, REFINE -> 0, 1, 2
        bf4_t x[6], a1[4], a2[4];
        f4_t z1[4], z2[4], z3;
        standardise(V, R, in, g, x);
        mlp_layers(W, V, g, x, z1, a1, z2, a2, z3);
        next = load_row(feat, row + stride, n, g);
        next_tag = row + stride < n ? tags[row + stride] : 0;
        // softmax cross-entropy of row li in the lanes g = 0
        f4_t d3 = zero;
        if (g == 0 && in) {
            const float zm = fmaxf(fmaxf(z3[0], z3[1]), z3[2]);
            float e[NOUT], se = 0.f;
#pragma unroll
            for (int j = 0; j < NOUT; ++j) {
                e[j] = expf(z3[j] - zm);
                se += e[j];
            }
            const float zl = lab == 0 ? z3[0] : (lab == 1 ? z3[1] : z3[2]);
            loss += -(zl - zm - logf(se));
#pragma unroll
            for (int j = 0; j < NOUT; ++j) d3[j] = (e[j] / se - (j == lab ? 1.f : 0.f)) * inv_n;
        }
        gb3 += d3;
        const bf4_t d3b = pack4(d3);
        // d2 = (W3^T d3) [z2 > 0], d1 = (W2^T d2) [z1 > 0]
        bf4_t d2b[4], d1b[4];
        f4_t d2[4], d1[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            d2[t] = mma(F.w3t[t][l], d3b, zero);
#pragma unroll
            for (int r = 0; r < 4; ++r) d2[t][r] = z2[t][r] > 0.f ? d2[t][r] : 0.f;
            gb2[t] += d2[t];
            d2b[t] = pack4(d2[t]);
            d1[t] = zero;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int t = 0; t < 4; ++t) d1[t] = mma(F.w2t[t][c][l], d2b[c], d1[t]);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
#pragma unroll
            for (int r = 0; r < 4; ++r) d1[t][r] = z1[t][r] > 0.f ? d1[t][r] : 0.f;
            gb1[t] += d1[t];
            d1b[t] = pack4(d1[t]);
        }
        if (trace && in) {
            float *tr = trace + row * MLP_TRACE;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
#pragma unroll
                for (int c = 0; c < 6; ++c)
                    if (16 * c + 4 * g + r < NIN) tr[16 * c + 4 * g + r] = bf2f((uint16_t)x[c][r]);
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int h = 16 * t + 4 * g + r;
                    tr[NIN + h] = bf2f((uint16_t)a1[t][r]);
                    tr[NIN + NH + h] = bf2f((uint16_t)a2[t][r]);
                    tr[NIN + 2 * NH + NOUT + h] = d2[t][r];
                    tr[NIN + 3 * NH + NOUT + h] = d1[t][r];
                }
                if (g == 0 && r < NOUT) tr[NIN + 2 * NH + r] = d3[r];
            }
        }
        // the operands of the weight gradients
        const int at = 16 * w + li;
#pragma unroll
        for (int c = 0; c < 6; ++c) put_block(S.x, 16 * c + 4 * g, at, x[c]);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            put_block(S.a1, 16 * t + 4 * g, at, a1[t]);
            put_block(S.a2, 16 * t + 4 * g, at, a2[t]);
            put_block(S.d1, 16 * t + 4 * g, at, d1b[t]);
            put_block(S.d2, 16 * t + 4 * g, at, d2b[t]);
        }
        put_block(S.d3, 4 * g, at, d3b);
        __syncthreads();
        // gW1 = d1 x^T, gW2 = d2 a1^T, gW3 = d3 a2^T over the pass's rows
#pragma unroll
        for (int k = 0; k < GROWS; k += 16) {
            const int h = 2 * k / GROWS;
            const bf4_t p1 = get_block(S.d1, 16 * ot + li, k + 4 * g), p2 = get_block(S.d2, 16 * ot + li, k + 4 * g);
#pragma unroll
            for (int c = 0; c < 3; ++c)
                gw1[h][c] = mma(p1, get_block(S.x, 16 * (3 * half + c) + li, k + 4 * g), gw1[h][c]);
#pragma unroll
            for (int c = 0; c < 2; ++c)
                gw2[h][c] = mma(p2, get_block(S.a1, 16 * (2 * half + c) + li, k + 4 * g), gw2[h][c]);
            if (half == 0)
                gw3[h] = mma(get_block(S.d3, li, k + 4 * g), get_block(S.a2, 16 * ot + li, k + 4 * g), gw3[h]);
        }
        __syncthreads();  // the operands are read before the next pass writes its own
    }
    // the bias gradients and the loss: over the 16 lanes of a group, then over the waves, in order
#pragma unroll
    for (int m = 1; m < 16; m <<= 1) {
        loss += __shfl_xor(loss, m);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            gb3[r] += __shfl_xor(gb3[r], m);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                gb1[t][r] += __shfl_xor(gb1[t][r], m);
                gb2[t][r] += __shfl_xor(gb2[t][r], m);
            }
        }
    }
    if (li == 0) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                bias[w][16 * t + 4 * g + r] = gb1[t][r];
                bias[w][NH + 16 * t + 4 * g + r] = gb2[t][r];
            }
        if (g == 0) {
#pragma unroll
            for (int j = 0; j < NOUT; ++j) bias[w][2 * NH + j] = gb3[j];
            bias[w][2 * NH + NOUT] = loss;
        }
    }
    float *out = part + (int64_t)blockIdx.x * (MLP_NPARAM + 1);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int o = 16 * ot + 4 * g + r;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const int i = 16 * (3 * half + c) + li;
            if (i < NIN) out[OW1 + o * NIN + i] = gw1[0][c][r] + gw1[1][c][r];
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) out[OW2 + o * NH + 16 * (2 * half + c) + li] = gw2[0][c][r] + gw2[1][c][r];
        if (half == 0 && 4 * g + r < NOUT) out[OW3 + (4 * g + r) * NH + 16 * ot + li] = gw3[0][r] + gw3[1][r];
    }
    __syncthreads();
    const int t = threadIdx.x;
    if (t < 2 * NH + NOUT + 1) {
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < GWAVES; ++k) s += bias[k][t];
        out[t < NH ? OB1 + t : (t < 2 * NH ? OB2 + t - NH : OB3 + t - 2 * NH)] = s;  // OB3 + NOUT is the loss
    }
}
static_assert(OB3 + NOUT == MLP_NPARAM, "the loss follows the last bias");

// Work-groups of the gradient kernel: one per CU, or one per pass where that is fewer.
constexpr int MLP_GRAD_BLOCKS = 256;

// grad[q] = the sum of the partials' column q (q = NPARAM: the loss, divided by n), in a fixed order:
// four threads take a quarter of the rows each, then the quarters are added.
__global__ __launch_bounds__(256) void k_mlp_reduce(const float *__restrict__ part, int32_t nblk, int64_t n,
                                                    float *__restrict__ grad, float *__restrict__ loss)
{
    __shared__ float quarter[4][64];
    const int q = blockIdx.x * 64 + (threadIdx.x & 63), k = threadIdx.x >> 6;
    const int b0 = nblk * k / 4, b1 = nblk * (k + 1) / 4;
    float s = 0.f;
    if (q <= MLP_NPARAM) {
#pragma unroll 8
        for (int b = b0; b < b1; ++b) s += part[(int64_t)b * (MLP_NPARAM + 1) + q];
    }
    quarter[k][threadIdx.x & 63] = s;
    __syncthreads();
    if (k == 0 && q <= MLP_NPARAM) {
        const int i = threadIdx.x;
        const float t = (quarter[0][i] + quarter[1][i]) + (quarter[2][i] + quarter[3][i]);
        if (q < MLP_NPARAM) grad[q] = t;
        else if (loss) *loss = t / (float)n;
    }
}

__global__ void k_mlp_adam(float *__restrict__ p, float *__restrict__ m, float *__restrict__ v,
                           const float *__restrict__ g, float lr, float b1, float b2, float eps, float c1, float c2)
{
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= MLP_NPARAM) return;
    const float gq = g[q];
    const float mq = b1 * m[q] + (1.f - b1) * gq;
    const float vq = b2 * v[q] + (1.f - b2) * gq * gq;
    m[q] = mq;
    v[q] = vq;
    p[q] -= lr * (mq / c1) / (sqrtf(vq / c2) + eps);
}

// Features: one work-group per patch, one thread per interior cell; the indicators are scaled
// by the patch spacing (dx |grad chi|, dx |grad alpha|, dx^2 |H|) like the plain criterion's.
__global__ __launch_bounds__(256) void k_features(const double *__restrict__ Q, const double *__restrict__ HM,
                                                  const PatchGeom *__restrict__ geom, float *__restrict__ feat)
{
    __shared__ double cellv[NCELL * 3];  // per interior cell: |grad chi|, |grad alpha|, |H|
    const int p = blockIdx.x, t = threadIdx.x;
    const PatchGeom g = geom[p];
    const double *qp = Q + (int64_t)p * PS;
    __shared__ double mx[27][3];
    if (t < 81) mx[t / 3][t % 3] = 0.0;
    for (int c = t; c < NCELL; c += blockDim.x) {
        const int x = c % 9 + 3, y = (c / 9) % 9 + 3, z = c / 81 + 3;
        const int o = boff(x, y, z);
        double gc = 0.0, ga = 0.0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int s = a == 0 ? 1 : (a == 1 ? YS : ZS);
            double wc[5], wa[5];
#pragma unroll
            for (int k = -2; k <= 2; ++k) {
                const double ph = qp[SPHI * CS + o + k * s];
                wc[k + 2] = ph * ph;
                wa[k + 2] = qp[SALPHA * CS + o + k * s];
            }
            const double i12 = 1.0 / (12.0 * g.dx[a]);
            const double dc = (8.0 * (wc[3] - wc[1]) - (wc[4] - wc[0])) * i12;
            const double da = (8.0 * (wa[3] - wa[1]) - (wa[4] - wa[0])) * i12;
            gc += dc * dc;
            ga += da * da;
        }
        cellv[3 * c + 0] = g.dx[0] * sqrt(gc);
        cellv[3 * c + 1] = g.dx[0] * sqrt(ga);
        cellv[3 * c + 2] = g.dx[0] * g.dx[0] * fabs(HM[((int64_t)p * 4 + 0) * NCELL + c]);
    }
    __syncthreads();
    if (t < 81) {
        const int b = t / 3, q = t % 3;
        const int bx = b % 3, by = (b / 3) % 3, bz = b / 9;
        double m = 0.0;
        for (int dz = 0; dz < 3; ++dz)
            for (int dy = 0; dy < 3; ++dy)
                for (int dx = 0; dx < 3; ++dx) {
                    const int c = ((3 * bz + dz) * 9 + 3 * by + dy) * 9 + 3 * bx + dx;
                    m = fmax(m, cellv[3 * c + q]);
                }
        feat[(int64_t)p * NIN + 3 * b + q] = (float)log10(m + 1e-12);
    }
}

// Learned tags, first pass: plain REFINE is kept; a confident learned REFINE is added (below
// max_level); a plain COARSEN survives unless the network is confident that the patch is not
// to be coarsened (pre = -1 marks the surviving candidates).
__global__ void k_tag_learned_pre(const float *__restrict__ logits, const int8_t *__restrict__ plain,
                                  const PatchGeom *__restrict__ geom, int32_t npatch, float conf, int32_t max_level,
                                  int8_t *__restrict__ pre)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= npatch) return;
    const float z0 = logits[3 * p], z1 = logits[3 * p + 1], z2 = logits[3 * p + 2];
    const float zm = fmaxf(fmaxf(z0, z1), z2);
    const float e0 = expf(z0 - zm), e1 = expf(z1 - zm), e2 = expf(z2 - zm);
    const float pm = 1.0f / (e0 + e1 + e2);  // probability of the arg-max class (its e is 1)
    const int cls = z2 >= zm ? 1 : (z1 >= zm ? 0 : -1);  // ties go to the higher class
    const bool sure = pm >= conf;
    int8_t tg = 0;
    if (plain[p] == 1) tg = 1;
    else if (sure && cls == 1 && geom[p].level < max_level) tg = 1;
    else if (plain[p] == -1 && !(sure && cls != -1)) tg = -1;
    pre[p] = tg;
}

// second pass: a family coarsens only if all 27 of its leaves are coarsening candidates
__global__ void k_tag_learned_family(const int8_t *__restrict__ pre, const int32_t *__restrict__ sib,
                                     int32_t npatch, int8_t *__restrict__ tags)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= npatch) return;
    int8_t tg = pre[p];
    if (tg == -1) {
        for (int n = 0; n < 27; ++n) {
            const int s = sib[(int64_t)p * 27 + n];
            if (s < 0 || pre[s] != -1) {
                tg = 0;
                break;
            }
        }
    }
    tags[p] = tg;
}

}  // namespace

int32_t mlp_tiles(int64_t n) { return (int32_t)((n + TILE - 1) / TILE); }

// Partial sums of the loss gradient for callers that cannot allocate a workspace: a
// file-scope device array, one copy per GPU, held until the process ends.  Its device address is
// taken once per device with hipGetSymbolAddress (the array's name is not a device address in
// host code) and kept; kernels receive that address.  Every grad call on a GPU shares the array.
__device__ __align__(256) float scratch[MLP_SCRATCH_TILES * (MLP_NPARAM + 1)];

hipError_t mlp_scratch(float **out)
{
    constexpr int MAXDEV = 64;
    static std::mutex mu;
    static float *addr[MAXDEV] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= MAXDEV) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[dev] = static_cast<float *>(ptr);
    }
    *out = addr[dev];
    return hipSuccess;
}

hipError_t launch_features(const double *Q, const double *HM, const PatchGeom *geom, int32_t npatch, float *feat,
                           hipStream_t st)
{
    if (npatch <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_features, dim3(npatch), dim3(256), 0, st, Q, HM, geom, feat);
    return hipGetLastError();
}

hipError_t launch_mlp_forward(const float *prm, const float *norm, const float *feat, int64_t n, float *logits,
                              hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    // waves of a few row blocks each once the chip is full (four work-groups per CU)
    const int64_t nb = std::min<int64_t>(mlp_tiles(n), 1024);
    hipLaunchKernelGGL(k_mlp_forward, dim3((unsigned)nb), dim3(256), 0, st, prm, norm, feat, n, logits);
    return hipGetLastError();
}

hipError_t launch_mlp_grad(const float *prm, const float *norm, const float *feat, const int8_t *tags, int64_t n,
                           float *work, float *trace, float *grad, float *loss, hipStream_t st)
{
    const int32_t nt = mlp_tiles(n), nb = std::min((nt + GROWS / TILE - 1) / (GROWS / TILE), MLP_GRAD_BLOCKS);
    if ((nt + 63) / 64 > 65535) return hipErrorInvalidConfiguration;  // more than 268 M rows are refused
    hipLaunchKernelGGL(k_mlp_grad, dim3(nb), dim3(64 * GWAVES), 0, st, prm, norm, feat, tags, n, work, trace);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_mlp_reduce, dim3((MLP_NPARAM + 1 + 63) / 64), dim3(256), 0, st, work, nb, n, grad, loss);
    return hipGetLastError();
}

hipError_t launch_mlp_adam(float *prm, float *m, float *v, const float *grad, float lr, float b1, float b2, float eps,
                           float c1, float c2, hipStream_t st)
{
    hipLaunchKernelGGL(k_mlp_adam, dim3((MLP_NPARAM + 255) / 256), dim3(256), 0, st, prm, m, v, grad, lr, b1, b2, eps,
                       c1, c2);
    return hipGetLastError();
}

hipError_t launch_tag_learned(const float *logits, const int8_t *plain, const PatchGeom *geom, const int32_t *sib,
                              int32_t npatch, float conf, int32_t max_level, int8_t *pre, int8_t *tags,
                              hipStream_t st)
{
    if (npatch <= 0) return hipSuccess;
    const unsigned nb = (unsigned)((npatch + 127) / 128);
    hipLaunchKernelGGL(k_tag_learned_pre, dim3(nb), dim3(128), 0, st, logits, plain, geom, npatch, conf, max_level,
                       pre);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_tag_learned_family, dim3(nb), dim3(128), 0, st, pre, sib, npatch, tags);
    return hipGetLastError();
}

}  // namespace ccz4
